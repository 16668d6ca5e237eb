"""Projected records at the edges of a wave (64 Gaussians): every record of every view written, none
past the end, culled ones as zeros (GPU only)."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2501_14534_amd import gs, raster, scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gs.load()


@pytest.mark.parametrize("n,deg", [(1, 0), (63, 1), (64, 3), (65, 2), (257, 3)])
def test_records_at_wave_edges(n, deg):
    from tests import parity as P
    wl = scenes.tiny(n=n, seed=n + 3, deg=deg, masks=True, band_masks=deg > 0)
    sc = wl.scene.copy()
    if n > 2:
        sc.means[0, 2] = np.nan          # culled: an input that is read is not finite
        sc.mask_logits[1] = np.inf
    if deg > 0 and n > 4:
        sc.sh_mask_logits[0, 3] = -4.0   # band off: its coefficients are not read
        sc.sh_rest[0, 0, 3] = np.nan
        sc.mask_logits[3] = 4.0
    cams = [wl.cams[0], dataclasses.replace(wl.cams[0], width=31, height=50)]
    wl = dataclasses.replace(wl, scene=sc, cams=cams)
    r = P.make_rasterizer(wl)
    r.splats.fill_(-7.0)
    extra = torch.full((2 * n * gs.SPLAT_FLOATS + 64,), -7.0, dtype=torch.float32, device="cuda")
    r.proj = gs.GsProjected(extra.data_ptr(), r.tiles_touched.data_ptr())
    r.project(raster.to_device(sc))
    torch.cuda.synchronize()
    print(f"[project] n {n} deg {deg}", flush=True)
    assert bool((extra[2 * n * gs.SPLAT_FLOATS:] == -7.0).all())
    r.splats[: 2 * n * gs.SPLAT_FLOATS] = extra[: 2 * n * gs.SPLAT_FLOATS]
    rec = r.splat_records()
    assert bool(((rec[:, 11] == 0) | (rec[:, 11] == 1)).all())
    assert bool((rec[rec[:, 11] == 0] == 0).all())
    if n > 2:
        assert float(rec[2, 11]) == 0.0 and float(rec[1, 11]) == 0.0
    if deg > 0 and n > 4:
        assert float(rec[3, 11]) == 1.0
        clean = sc.copy()
        clean.sh_rest[0, 0, 3] = 0.0     # the oracle multiplies a masked band by zero
        wl = dataclasses.replace(wl, scene=clean)
    P.check_projection(wl, wl.opts, r)
