"""The forward walk's slices of a list and its groups of records (GPU only): slices of one entry, of
a power of two below the batch depth, of a chunk; lists of every length around a slice and a group."""
import dataclasses

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_14534_amd import gs
    gs.load()


def _run(wl, opts, dL):
    from tests import parity as P
    r, params = P.gpu_forward(wl, opts)
    grads = r.zero_grads(params)
    r.backward(params, dL, grads)
    hits = torch.zeros(wl.scene.n, dtype=torch.int32, device="cuda")
    r.count_hits(hits)
    torch.cuda.synchronize()
    return r, grads, hits


@pytest.mark.parametrize("batch,bwd_chunk,ppt,cull", [
    (1, 64, 1, 1), (3, 64, 1, 1), (63, 16, 1, 1), (65, 128, 1, 0), (128, 0, 1, 1), (1024, 32, 2, 1), (63, 64, 4, 1)])
def test_slice_sizes_give_the_same_image_and_hits(batch, bwd_chunk, ppt, cull):
    """Pixels stop inside groups of four, two and one: image, transmittance, last contributor and hits
    bit for bit, gradients within the tolerance of the layouts test."""
    from tests.test_gpu_blocks import _workload
    from tests.test_gpu_edges import _rel_close
    wl = _workload()
    dL = torch.from_numpy(np.random.default_rng(5).standard_normal(3 * 203 * 139).astype(np.float32) * 1e-3).cuda()
    ref, gref, href = _run(wl, wl.opts, dL)
    print(f"[slices] batch {batch} chunk {bwd_chunk} ppt {ppt} cull {cull}", flush=True)
    tile = {1: (16, 16), 2: (32, 16), 4: (32, 32)}[ppt]
    r, g, h = _run(wl, dataclasses.replace(wl.opts, batch_depth=batch, bwd_chunk=bwd_chunk, pixels_per_thread=ppt,
                                           subtile_cull=cull, tile_w=tile[0], tile_h=tile[1]), dL)
    assert torch.equal(r.image, ref.image) and torch.equal(r.T_final, ref.T_final)
    assert torch.equal(h, href)
    if ppt == 1:
        assert torch.equal(r.last, ref.last)
    keep = torch.arange(wl.scene.n, device="cuda") != 5  # the giant's gradients are rounding alone
    for k in g:
        assert _rel_close(g[k][..., keep], gref[k][..., keep], 1e-3), k


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 63, 64, 65, 127, 128, 129, 131, 193])
def test_lists_around_a_slice_and_a_group(n):
    """n faint Gaussians, all over every pixel of one 8 x 8 view: each is hit by every pixel, and the
    image is that of slices of one entry."""
    from paper_2501_14534_amd import scenes
    wl = scenes.tiny(n=n, seed=n, deg=0, width=8, height=8, log_scale=(1.5, 0.0), opacity=(-4.0, 0.0))
    dL = torch.ones(3 * 64, device="cuda")
    print(f"[slices] n {n}", flush=True)
    a, ga, ha = _run(wl, wl.opts, dL)
    b, gb, hb = _run(wl, dataclasses.replace(wl.opts, batch_depth=1), dL)
    assert torch.equal(a.image, b.image) and torch.equal(a.last, b.last) and torch.equal(ha, hb)
    assert int(a.last.max()) == n or int(ha.min()) == 0  # every list is walked to its end
    assert int(ha.sum()) > 0
