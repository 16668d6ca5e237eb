"""Two records in one reduction of the backward walk (GPU only): a record's row does not depend on
whether, or with which record, it shares the reduction."""
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


@pytest.mark.parametrize("n", [1, 2, 3, 64, 65, 400])
@pytest.mark.parametrize("tw,th,ppt,cull", [(8, 8, 1, 1), (16, 16, 1, 0), (32, 16, 2, 1), (32, 32, 4, 1)])
def test_rows_do_not_depend_on_the_pairing(n, tw, th, ppt, cull):
    """Batches of one entry (never two records), of 7 (an odd one left over) and of the default depth
    give the same rows bit for bit."""
    wl = scenes.tiny(n=n, seed=n, deg=0, width=67, height=41, log_scale=(-1.8, 0.8), opacity=(0.0, 1.5))
    params = raster.to_device(wl.scene)
    dL = torch.from_numpy(np.random.default_rng(6).standard_normal(3 * 67 * 41).astype(np.float32)).cuda()
    print(f"[pairs] n {n} tile {tw}x{th} ppt {ppt} cull {cull}", flush=True)
    rows = []
    for batch in (wl.opts.batch_depth, 7, 1):
        r = raster.Rasterizer(n, 0, wl.cams, dataclasses.replace(
            wl.opts, tile_w=tw, tile_h=th, pixels_per_thread=ppt, subtile_cull=cull, batch_depth=batch))
        r.forward(params)
        rows.append(r.grad_pairs(dL).clone())
    assert float(rows[0].abs().max()) > 0.0
    assert torch.equal(rows[0], rows[1]) and torch.equal(rows[0], rows[2])
