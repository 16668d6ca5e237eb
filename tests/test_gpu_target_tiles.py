"""The tiles of the target blur and the stretches of the resize at their edges (GPU only), against
the double-precision oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("k,sigma", [(1, 1.0), (3, 0.7), (5, 1.2), (9, 2.4), (15, 3.0), (31, 6.0)])
def test_blur_tiles(k, sigma):
    """Widths and heights one pixel less, exactly and one pixel more than the tile of that radius, and
    images smaller than the radius.  Two passes of k products of values in [0, 1] with weights that
    sum to one: |error| <= 2 k 2^-24."""
    from oracle import targets as TG
    from paper_2501_14534_amd import progressive as PG
    from tests.test_gpu_progressive import _cams, _split
    tw = 128 - (k + 2) // 4 * 4
    cams = _cams([(tw - 1, 15), (tw, 16), (tw + 1, 17), (2 * tw, 31), (2 * tw + 2, 8), (3, 40), (1, 1)])
    rng = np.random.default_rng(k)
    img = rng.random(sum(3 * c.width * c.height for c in cams)).astype(np.float32)
    print(f"[blur tiles] k={k}", flush=True)
    got = PG.blur(torch.from_numpy(img).cuda(), cams, k, sigma).cpu().numpy()
    ref = TG.blur_views(_split(img.astype(np.float64), cams), k, sigma)
    assert np.abs(got - np.concatenate([r.reshape(-1) for r in ref])).max() <= 2 * k * 2.0 ** -24 + 2.0 ** -23


@pytest.mark.parametrize("src,dst", [
    ((2100, 9), (2, 2)), ((1500, 3), (1, 1)), ((3000, 5), (700, 3)), ((1023, 4), (1022, 4)), ((40, 7), (513, 20)),
    ((1, 300), (1, 7)), ((1026, 2), (1, 1)), ((256, 2), (256, 2))])
def test_resize_stretches(src, dst):
    """One output over more columns than a workgroup stages, several stretches of a row, more outputs
    than inputs, one column.  A float sum of the box's columns, then rows: |error| <= (bw + bh + 3) 2^-24."""
    from oracle import targets as TG
    from paper_2501_14534_amd import progressive as PG
    from tests.test_gpu_progressive import _cams, _split
    cams, out = _cams([src, (33, 5), src]), _cams([dst, (7, 5), dst])
    rng = np.random.default_rng(src[0])
    img = rng.random(sum(3 * c.width * c.height for c in cams)).astype(np.float32)
    print(f"[resize stretches] {src} -> {dst}", flush=True)
    got = PG.resize(torch.from_numpy(img).cuda(), cams, out).cpu().numpy()
    ref = TG.resize_views(_split(img.astype(np.float64), cams), [(c.width, c.height) for c in out])
    terms = -(-src[0] // dst[0]) - (-src[1] // dst[1]) + 2 + 5 + 3
    assert np.abs(got - np.concatenate([r.reshape(-1) for r in ref])).max() <= terms * 2.0 ** -24
