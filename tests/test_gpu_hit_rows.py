"""The backward walk keeps rows only for the pairs that some pixel composites, unless the rows are
the caller's (GPU only): batches with a tail, of one entry, of several 64-entry chunks."""
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


@pytest.mark.parametrize("batch,tw,th,ppt,cull", [
    (1, 16, 16, 1, 1), (63, 16, 16, 1, 1), (64, 16, 16, 1, 0), (100, 16, 16, 2, 1), (129, 32, 32, 4, 1),
    (1024, 8, 8, 1, 1), (100, 32, 16, 2, 0)])
def test_rows_of_composited_pairs(batch, tw, th, ppt, cull):
    """Every pair in front of its tile's last contributor has its row in the caller's buffer, zero
    where no pixel composites it; the gradients (over the kept rows) are the sums of those rows:
    half a unit in the last place, plus the double sum's own rounding."""
    n = 500
    wl = scenes.tiny(n=n, seed=21, deg=1, width=203, height=139, log_scale=(-2.2, 1.0), opacity=(1.0, 1.5))
    opts = dataclasses.replace(wl.opts, tile_w=tw, tile_h=th, pixels_per_thread=ppt, subtile_cull=cull,
                               batch_depth=batch, bwd_chunk=64)
    print(f"[rows] batch {batch} tile {tw}x{th} ppt {ppt} cull {cull}", flush=True)
    params = raster.to_device(wl.scene)
    r = raster.Rasterizer(n, 1, wl.cams, opts)
    r.forward(params)
    dL = torch.from_numpy(np.random.default_rng(4).standard_normal(3 * r.total_pixels).astype(np.float32)).cuda()
    mean2d = torch.zeros(2 * n, dtype=torch.float32, device="cuda")
    r.backward(params, dL, r.zero_grads(params), mean2d)
    gp = torch.full((r.capacity * 9,), float("nan"), device="cuda")
    r.blend_bwd(dL, gp)
    rows = gp[: r.pairs() * 9].view(-1, 9)
    written = ~rows.isnan().any(1)
    assert bool(rows[~written].isnan().all())
    zero = (rows == 0).all(1)
    assert int(zero.sum()) > 0 and int((~zero & written).sum()) > 0
    # walked: up to the largest last_contrib of the tile (list positions from 1)
    W, H = 203, 139
    TX, TY = -(-W // tw), -(-H // th)
    last = torch.zeros(TY * th, TX * tw, dtype=torch.int64, device="cuda")
    last[:H, :W] = r.last.view(H, W).long()
    most = last.view(TY, th, TX, tw).amax((1, 3)).flatten()
    rg = r.ranges.long().view(-1, 2)[: TX * TY]
    pos = torch.arange(r.pairs(), device="cuda")
    tile = torch.bucketize(pos, rg[:, 1].cummax(0).values, right=True)
    walked = torch.zeros(r.pairs(), dtype=torch.bool, device="cuda")
    walked[r.pair_index[: r.pairs()].long()] = pos < (rg[:, 0] + most)[tile]
    assert torch.equal(written, walked)
    owner = torch.repeat_interleave(torch.arange(n, device="cuda"), r.tiles_touched[:n].long())
    d = rows.nan_to_num(0.0).double()
    ref = torch.zeros(n, 9, dtype=torch.float64, device="cuda").index_add_(0, owner, d)
    mag = torch.zeros(n, 9, dtype=torch.float64, device="cuda").index_add_(0, owner, d.abs())
    for k in range(2):
        err = (mean2d[k * n:(k + 1) * n].double() - ref[:, k]).abs()
        assert bool((err <= 2.0 ** -24 * ref[:, k].abs() + 1e-12 * mag[:, k]).all())
