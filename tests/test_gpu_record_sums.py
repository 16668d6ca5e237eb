"""Per-record sums of the pair gradients and the packed records that the projection backward works on
(GPU only): short, long and heavy records, and both splits of the views over the waves."""
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


@pytest.mark.parametrize("n", [1, 63, 64, 65, 700])
def test_sums_of_short_long_and_heavy_records(n):
    """mean2d receives the sums of the (u, v) columns: each within half a unit in the last place of
    the double sum of its rows (plus the double sum's own rounding)."""
    wl = scenes.tiny(n=n, seed=n, deg=1, width=203, height=139, log_scale=(-2.2, 1.3), opacity=(-1.0, 1.0))
    opts = dataclasses.replace(wl.opts, tile_w=8, tile_h=8, bwd_chunk=64)
    params = raster.to_device(wl.scene)
    r = raster.Rasterizer(n, 1, wl.cams, opts)
    r.forward(params)
    dL = torch.from_numpy(np.random.default_rng(1).standard_normal(3 * r.total_pixels).astype(np.float32)).cuda()
    mean2d = torch.zeros(2 * n, dtype=torch.float32, device="cuda")
    r.backward(params, dL, r.zero_grads(params), mean2d)
    rows = r.grad_pairs(dL).double()
    owner = torch.repeat_interleave(torch.arange(n, device="cuda"), r.tiles_touched[:n].long())
    print(f"[sums] n {n}: pairs per record up to {int(r.tiles_touched[:n].max())}", flush=True)
    if n == 700:
        tt = r.tiles_touched[:n]
        assert int((tt > 256).sum()) > 0 and int(((tt > 96) & (tt <= 256)).sum()) > 0
    ref = torch.zeros(n, 9, dtype=torch.float64, device="cuda").index_add_(0, owner, rows)
    mag = torch.zeros(n, 9, dtype=torch.float64, device="cuda").index_add_(0, owner, rows.abs())
    for k in range(2):
        err = (mean2d[k * n:(k + 1) * n].double() - ref[:, k]).abs()
        assert bool((err <= 2.0 ** -24 * ref[:, k].abs() + 1e-12 * mag[:, k]).all())


@pytest.mark.parametrize("n,views", [(180_000, 6), (200_001, 7)])
def test_many_waves_give_the_per_view_gradients(n, views):
    """Enough waves for several views per wave (a remainder of views among them): bit for bit the
    gradients of the per-view calls, which take one view per wave."""
    wl = scenes.config(4, n=n)
    cams = [scenes.make_camera((8 * np.cos(t), 8 * np.sin(t), 0.5), (0, 0, 0), 96 + 8 * k, 72, 130.0)
            for k, t in enumerate(np.linspace(0, 5, views))]
    params = raster.to_device(wl.scene)
    assert (n + 63) // 64 * views > 4 * 4096 > (n + 63) // 64
    print(f"[sums] n {n}, {views} views", flush=True)

    def grads(cs, dL, g):
        r = raster.Rasterizer(n, 3, cs, wl.opts, mask_eps=wl.scene.mask_eps, sh_mask_eps=wl.scene.sh_mask_eps)
        r.forward(params)
        r.backward(params, dL, g)
        return r

    px = [3 * c.width * c.height for c in cams]
    dL = torch.from_numpy(np.random.default_rng(2).standard_normal(sum(px)).astype(np.float32) * 1e-3).cuda()
    r = raster.Rasterizer(n, 3, cams, wl.opts)
    ga, gb = r.zero_grads(params), r.zero_grads(params)
    grads(cams, dL, ga)
    for c, part in zip(cams, dL.split(px)):
        grads([c], part.contiguous(), gb)
    for k in ga:
        assert torch.equal(ga[k], gb[k]), k
        assert float(ga[k].abs().max()) > 0.0, k
