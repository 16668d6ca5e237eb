"""The loss's 116 x 16 tiles at their edges (GPU only): images of one pixel, a tile less, exact and
more in each direction, rows that start at any float's address, and a call whose tiles do not divide
by eight."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes", [
    [(1, 1)], [(115, 15), (116, 16), (117, 17)], [(232, 33), (233, 8), (5, 250)], [(119, 7), (1, 40), (350, 1)],
    [(118, 24)]])
def test_tile_edges(sizes):
    """Against the double-precision oracle, with the tolerances of the loss tests."""
    from paper_2501_14534_amd.photometric import PhotometricLoss
    from tests.test_gpu_loss import _cams, _check
    cams = _cams(sizes)
    rng = np.random.default_rng(17)
    n = sum(3 * w * h for w, h in sizes)
    img = rng.random(n).astype(np.float32)
    tgt = rng.random(n).astype(np.float32)
    tgt[::89] = img[::89]
    print(f"[loss] {sizes}", flush=True)
    pl, ti, tt, loss, dL = _check(cams, img, tgt, 0.2)
    # each view alone gives the same gradient (of the mean over one view) as in the call of several
    o = 0
    for v, ((w, h), c) in enumerate(zip(sizes, cams)):
        k = 3 * w * h
        l1, d1 = PhotometricLoss([c], 0.2)(ti[o:o + k].contiguous(), tt[o:o + k].contiguous())
        assert float(l1[0]) == float(np.float32(loss[v]))
        d = torch.from_numpy(dL[o:o + k]).cuda() * len(sizes)
        assert bool(((d1 - d).abs() <= 4e-7 * d1.abs()).all())
        o += k
