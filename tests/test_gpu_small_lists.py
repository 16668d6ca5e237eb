"""The one-workgroup lists of small calls against the general path (GPU only): both sides of the
boundaries of 8192 and 12288 records, ties and equal depths, nothing visible, overflow; and a tile sort on both
sides of the block count up to which each block sums the histogram."""
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


@pytest.mark.parametrize("n,views,levels", [
    (1, 1, None), (64, 1, 1), (1024, 1, 3), (1025, 2, None), (4096, 2, None), (8191, 1, 5), (8192, 1, None),
    (2048, 4, None), (8193, 1, 5), (4096, 3, None), (12288, 1, None), (12289, 1, None)])
def test_lists_on_both_sides_of_the_boundary(n, views, levels):
    """Against the oracle's lists, word for word; the same Gaussians with invisible ones behind them,
    over 12288 records, take the general path and give the same lists."""
    from tests import parity as P
    wl = scenes.tiny(n=n, seed=n + views, deg=0, width=320, height=208, log_scale=(-3.6, 0.6), depth_levels=levels)
    cams = [dataclasses.replace(wl.cams[0], width=320 - 37 * v, height=208 - 21 * v) for v in range(views)]
    wl = dataclasses.replace(wl, cams=cams)
    print(f"[small lists] n {n}, {views} views, {levels} depths", flush=True)
    r, params = P.gpu_forward(wl)
    P.check_binning(wl, wl.opts, r)
    pad = 13000
    big = {k: torch.cat([v, torch.zeros(*v.shape[:-1], pad, device="cuda")], -1).contiguous()
           for k, v in params.items() if v is not None}
    big["means"][1, n:] = -5.0  # behind the camera
    q = raster.Rasterizer(n + pad, 0, cams, wl.opts)
    q.forward({**{k: None for k in params}, **big})
    K = r.pairs()
    assert q.pairs() == K and torch.equal(q.ranges, r.ranges)
    assert torch.equal(q.pair_index[:K], r.pair_index[:K])
    a, b = q.ids[:K].long(), r.ids[:K].long()
    assert torch.equal(a % (n + pad), b % n) and torch.equal(a // (n + pad), b // n)
    assert torch.equal(q.image, r.image)


def test_nothing_visible_and_overflow():
    wl = scenes.tiny(n=700, seed=1, deg=0, width=320, height=208)
    params = raster.to_device(wl.scene)
    r = raster.Rasterizer(700, 0, wl.cams, wl.opts)
    r.forward(params)
    K = r.pairs()
    behind = dict(params, means=params["means"].clone())
    behind["means"][1] = -5.0
    r.forward(behind)
    assert r.pairs() == 0 and not r.overflowed() and int(r.ranges.abs().max()) == 0
    q = raster.Rasterizer(700, 0, wl.cams, wl.opts, capacity=K - 1)
    q.project(params)
    q.bin_sort()
    assert q.overflowed() and q.pairs() == K and int(q.ranges.abs().max()) == 0


@pytest.mark.parametrize("capacity", [64 * 4096, 64 * 4096 + 1])
def test_histogram_rows_summed_by_the_blocks(capacity):
    from tests import parity as P
    wl = scenes.tiny(n=9000, seed=8, deg=0, width=600, height=410, log_scale=(-3.6, 0.6))
    print(f"[small lists] capacity {capacity}", flush=True)
    r, _ = P.gpu_forward(wl, capacity=capacity)
    assert r.capacity == capacity and not r.overflowed()
    P.check_binning(wl, wl.opts, r)
