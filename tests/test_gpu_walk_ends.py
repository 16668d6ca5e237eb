"""Every entry of a list is walked, forward, counting and backward (GPU only)."""
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


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 127, 128, 129, 192, 193, 197])
@pytest.mark.parametrize("tw,th,ppt,batch,chunk", [(16, 16, 1, 128, 256), (16, 16, 1, 1, 16), (16, 16, 2, 64, 64),
                                                   (16, 16, 4, 128, 0)])
def test_no_entry_is_left_out(n, tw, th, ppt, batch, chunk):
    """n faint Gaussians, each over every pixel of one 8 x 8 view and none opaque enough to stop one:
    each is hit by all 64 pixels, is the last contributor of all if it is the last, and gets the
    gradient of its (unclamped) colour; the transmittance is the product over all of them (2 n roundings)."""
    from tests import parity as P
    wl = scenes.tiny(n=n, seed=n, deg=0, width=8, height=8, log_scale=(3.0, 0.0), opacity=(-4.0, 0.0))
    opts = dataclasses.replace(wl.opts, tile_w=tw, tile_h=th, pixels_per_thread=ppt, batch_depth=batch, bwd_chunk=chunk)
    print(f"[walk ends] n {n} ppt {ppt} batch {batch} chunk {chunk}", flush=True)
    r, _ = P.gpu_forward(wl, opts)
    hits = torch.zeros(n, dtype=torch.int32, device="cuda")
    r.count_hits(hits)
    rows = r.grad_records(torch.ones(3 * 64, device="cuda"))
    torch.cuda.synchronize()
    assert (hits == 64).all() and (r.last == n).all()
    assert (rows[:, 6:9] > 0).all()
    rec = r.splat_records().cpu().numpy().astype(np.float64)
    y, x = np.meshgrid(np.arange(8) + 0.5, np.arange(8) + 0.5, indexing="ij")
    dx, dy = x[None] - rec[:, 0, None, None], y[None] - rec[:, 1, None, None]
    q = rec[:, 2, None, None] * dx * dx + 2 * rec[:, 3, None, None] * dx * dy + rec[:, 4, None, None] * dy * dy
    T = np.prod(1.0 - rec[:, 5, None, None] * np.exp(-0.5 * q), 0)
    assert np.abs(r.T_final.cpu().numpy().reshape(8, 8) / T - 1.0).max() <= (2 * n + 4) * 2.0 ** -24
