"""Both sides of the rule that chooses between a thread per output value and a workgroup per stretch of
an output row (GPU only), against the double-precision oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("views", [
    [((64, 48), (64, 48))], [((64, 48), (32, 24))], [((64, 48), (8, 6))], [((65, 47), (9, 7))],
    [((333, 250), (148, 111))], [((333, 250), (95, 71))], [((800, 300), (267, 100))], [((800, 300), (100, 37))],
    [((3, 3000), (3, 1500))], [((16, 2000), (2, 250))], [((2000, 16), (250, 2))], [((40, 30), (97, 61))],
    [((700, 500), (40, 30)), ((50, 40), (50, 40)), ((33, 21), (70, 50))],
    [((64, 48), (64, 48)), ((120, 90), (60, 45)), ((5, 4), (1, 1))]])
def test_resize_either_way(views):
    """Float sums of a box's rows and columns, in either order: |error| <= (bw + bh + 6) 2^-24 of values in
    [0, 1] with weights that sum to one (as many roundings as a box has rows and columns, a product each way,
    the division)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import targets as TG
    from paper_2501_14534_amd import progressive as PG
    from tests.test_gpu_progressive import _cams, _split
    cams, out = _cams([s for s, _ in views]), _cams([d for _, d in views])
    img = np.random.default_rng(views[0][0][0]).random(sum(3 * c.width * c.height for c in cams)).astype(np.float32)
    print(f"[resize rule] {views}", flush=True)
    got = PG.resize(torch.from_numpy(img).cuda(), cams, out).cpu().numpy()
    ref = TG.resize_views(_split(img.astype(np.float64), cams), [(c.width, c.height) for c in out])
    terms = max(-(-s[0] // d[0]) - (-s[1] // d[1]) + 2 for s, d in views) + 6
    assert np.abs(got - np.concatenate([r.reshape(-1) for r in ref])).max() <= terms * 2.0 ** -24
