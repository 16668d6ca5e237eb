"""Rows whose last tile would keep few columns are cut into about equal tiles (GPU only): widths on
both sides of that rule, against the double-precision oracles."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes", [[(132, 9), (133, 9)], [(128, 20), (116, 3), (248, 17), (249, 5)],
                                   [(3481, 5), (3496, 4), (3497, 4)]])
def test_loss_tiles(sizes):
    """Tolerances of the loss tests; 31 tiles of a row with one column left over."""
    from tests.test_gpu_loss import _cams, _check
    rng = np.random.default_rng(23)
    n = sum(3 * w * h for w, h in sizes)
    img = rng.random(n).astype(np.float32)
    print(f"[even tiles] loss {sizes}", flush=True)
    _check(_cams(sizes), img, rng.random(n).astype(np.float32), 0.2)


@pytest.mark.parametrize("k,sigma", [(1, 1.0), (7, 1.5), (31, 6.0)])
def test_blur_tiles(k, sigma):
    """16 and 17 columns left over, one and 30 tiles before them.  |error| <= 2 k 2^-24 (two passes of k
    products of values in [0, 1], weights that sum to one) and the result's rounding."""
    from oracle import targets as TG
    from paper_2501_14534_amd import progressive as PG
    from tests.test_gpu_progressive import _cams, _split
    tw = 128 - (k + 2) // 4 * 4
    cams = _cams([(tw + 16, 17), (tw + 17, 5), (30 * tw + 1, 3), (30 * tw + 16, 3), (2 * tw + 3, 18)])
    img = np.random.default_rng(k).random(sum(3 * c.width * c.height for c in cams)).astype(np.float32)
    print(f"[even tiles] blur k={k}", flush=True)
    got = PG.blur(torch.from_numpy(img).cuda(), cams, k, sigma).cpu().numpy()
    ref = TG.blur_views(_split(img.astype(np.float64), cams), k, sigma)
    assert np.abs(got - np.concatenate([r.reshape(-1) for r in ref])).max() <= 2 * k * 2.0 ** -24 + 2.0 ** -23
