"""Four elements a thread of gs_l2_grad at the ends of views (GPU only): views of 3 to 45 elements,
several inside one quad, buffers at every word of a 16-byte line."""
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


@pytest.mark.parametrize("sizes", [[(1, 1)], [(1, 1)] * 5, [(5, 3), (1, 1), (7, 1), (2, 2)], [(343, 1), (1, 1)]])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
def test_ends_of_views(sizes, shift):
    """The same single-precision operations element by element: equal bit for bit."""
    from paper_2501_14534_amd import gs
    cams = [scenes.make_camera([0, -4, 0], [0, 0, 0], w, h, 4.0) for w, h in sizes]
    n = [3 * w * h for w, h in sizes]
    rng = np.random.default_rng(shift)
    img, tgt = rng.random(sum(n)).astype(np.float32), rng.random(sum(n)).astype(np.float32)
    print(f"[l2 quads] {sizes} shift {shift}", flush=True)
    a, b = torch.zeros(sum(n) + shift, device="cuda"), torch.zeros(sum(n) + shift, device="cuda")
    a[shift:] = torch.from_numpy(img).cuda()
    b[shift:] = torch.from_numpy(tgt).cuda()
    out = torch.full((sum(n) + shift + 4,), float("nan"), device="cuda")
    gs.check(gs.l2_grad(a.data_ptr() + 4 * shift, b.data_ptr() + 4 * shift, gs.cameras(cams), len(cams), len(cams),
                        out.data_ptr() + 4 * shift, torch.cuda.current_stream().cuda_stream), "gs_l2_grad")
    got = out.cpu().numpy()
    scale = np.concatenate([np.full(k, np.float32(2.0 / (k * len(cams))), np.float32) for k in n])
    np.testing.assert_array_equal(got[shift:shift + sum(n)], scale * (img - tgt))
    assert np.isnan(got[shift + sum(n):]).all() and np.isnan(got[:shift]).all()
