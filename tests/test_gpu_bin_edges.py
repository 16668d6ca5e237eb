"""Lists around the block sizes of the binning: records per scan block (1024, 4096), output positions per
emission chunk (4096), records larger than a chunk, one and many tile digits (GPU only)."""
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


@pytest.mark.parametrize("n,views,tile,log_scale", [
    (1, 1, 8, -1.0), (63, 2, 16, -3.0), (1023, 1, 8, -3.0), (1024, 1, 8, -3.0), (1025, 3, 16, -4.0),
    (4096, 1, 16, -4.0), (4097, 2, 8, -3.5), (9000, 3, 8, -4.5), (40, 1, 8, 1.5)])
def test_lists_are_exact(n, views, tile, log_scale):
    from tests import parity as P
    wl = scenes.tiny(n=n, seed=n, deg=0, width=600, height=410, log_scale=(log_scale, 0.6), masks=n % 2 == 1)
    cams = [dataclasses.replace(wl.cams[0], width=600 - 37 * v, height=410 - 21 * v) for v in range(views)]
    wl = dataclasses.replace(wl, cams=cams)
    opts = dataclasses.replace(wl.opts, tile_w=tile, tile_h=tile)
    r, _ = P.gpu_forward(wl, opts)
    K = r.pairs()
    print(f"[bin] n {n}, {views} views, tile {tile}: {K} pairs, {r.total_tiles} tiles", flush=True)
    if log_scale > 1.0:
        assert int(r.tiles_touched.max()) > 3800  # a record about a chunk long, or longer
    P.check_binning(wl, opts, r)
    # canonical positions: every pair once, and each pair's row inside its record's run
    idx = np.sort(r.pair_index[:K].cpu().numpy().view(np.uint32))
    np.testing.assert_array_equal(idx, np.arange(K, dtype=np.uint32))
    ids = r.ids[:K].long()
    off = r.offsets[ids].long() & 0xFFFFFFFF
    pos = r.pair_index[:K].long() - off
    assert bool(((pos >= 0) & (pos < r.tiles_touched[ids].long())).all())


def test_full_lists_and_one_pair_too_many():
    """A capacity of exactly K holds the lists; one less reports K and writes none."""
    from tests import parity as P
    wl = scenes.tiny(n=3000, seed=5, deg=0, width=320, height=240)
    K = P.gpu_forward(wl)[0].pairs()
    r, _ = P.gpu_forward(wl, capacity=K)
    assert r.capacity == K and not r.overflowed()
    P.check_binning(wl, wl.opts, r)
    from paper_2501_14534_amd import raster
    q = raster.Rasterizer(3000, 0, wl.cams, wl.opts, capacity=K - 1)
    q.project(raster.to_device(wl.scene))
    q.bin_sort()
    assert q.overflowed() and q.pairs() == K
    assert int(q.ranges.abs().max()) == 0
