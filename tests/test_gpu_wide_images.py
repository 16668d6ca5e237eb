"""Target images at the largest widths that a camera can state (GPU only; up to 156 GB of planes)."""
import numpy as np
import pytest
import torch

from paper_2501_14534_amd import gs, scenes

pytestmark = pytest.mark.gpu

INT_MAX = 2 ** 31 - 1


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GB of free device memory")
    gs.load()
    yield
    torch.cuda.empty_cache()


def _cams(w):
    return gs.cameras([scenes.Camera(np.eye(3, dtype=np.float32), np.zeros(3, np.float32), 1.0, 1.0, 0.0, 0.0, w, 1)])


@pytest.mark.parametrize("w,wo", [(INT_MAX, 1000003), (INT_MAX, 1000), (INT_MAX - 512, 999), (8, INT_MAX)])
def test_resize_to_and_from_the_widest_rows(w, wo):
    """Planes of 1, 2 and 3: a box of n equal values is off by at most n roundings."""
    src = torch.empty(3, w, device="cuda")
    for c in range(3):
        src[c] = c + 1
    out = torch.full((3, wo), -1.0, device="cuda")
    print(f"[wide] resize {w} -> {wo}", flush=True)
    gs.check(gs.resize_views(src.data_ptr(), _cams(w), out.data_ptr(), _cams(wo), 1,
                             torch.cuda.current_stream().cuda_stream), "gs_resize_views")
    torch.cuda.synchronize()
    tol = (w // wo + 2) * 2.0 ** -24
    for c in range(3):
        lo, hi = float(out[c].min()), float(out[c].max())
        assert (c + 1) * (1 - tol) <= lo and hi <= (c + 1) * (1 + tol), (c, lo, hi)


@pytest.mark.parametrize("w,h", [(1, 100_000_007), (1, INT_MAX), (INT_MAX, 1)])
def test_loss_of_the_longest_images(w, h):
    """One column or row, of more tiles than a launch is wide, up to the largest int: a uniform image
    against a uniform target.  Away from the ends every gradient is that of a line of 1000 pixels, scaled by
    the pixels' number (the window's taps and a quotient: a relative 2^-20), in every plane from the first
    tile to the last."""
    from paper_2501_14534_amd.photometric import PhotometricLoss
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 76 * w * h + (8 << 30):
        pytest.skip("not enough device memory")
    grads = []
    for n in (1000, w * h):
        cam = scenes.Camera(np.eye(3, dtype=np.float32), np.zeros(3, np.float32), 1.0, 1.0, 0.0, 0.0, n if w > 1 else 1,
                            n if h > 1 else 1)
        image, target = torch.full((3 * n,), 0.25, device="cuda"), torch.full((3 * n,), 0.75, device="cuda")
        out = torch.full((3 * n,), float("nan"), device="cuda")
        print(f"[wide] loss {cam.width} x {cam.height}", flush=True)
        loss, _ = PhotometricLoss([cam])(image, target, out=out)
        torch.cuda.synchronize()
        assert np.isfinite(float(loss[1]))
        for c in range(3):
            inner = out[c * n + 16:(c + 1) * n - 16]
            grads += [float(inner.min()) * n, float(inner.max()) * n]
    assert np.abs(np.array(grads) / grads[0] - 1.0).max() <= 2.0 ** -20, grads


@pytest.mark.parametrize("w", [2 ** 30 + 1, 2 ** 30 + 2, INT_MAX])
def test_blur_reflects_at_the_ends_of_the_widest_rows(w):
    """Zeros but for 1 .. 8 from either end of a row: with 7 taps the 5 values at either end are those of
    the row's first 16 values alone, and the middle is zero."""
    r, k, sigma = 3, 7, 1.5
    src = torch.zeros(3, w, device="cuda")
    ramp = torch.arange(1, 9, device="cuda", dtype=torch.float32)
    src[:, :8] = ramp
    src[:, -8:] = ramp.flip(0)
    small = torch.zeros(3, 16, device="cuda")
    small[:, :8] = ramp
    out, ref = torch.full((3, w), -1.0, device="cuda"), torch.empty(3, 16, device="cuda")
    print(f"[wide] blur {w}", flush=True)
    s = torch.cuda.current_stream().cuda_stream
    gs.check(gs.blur_views(small.data_ptr(), ref.data_ptr(), _cams(16), 1, k, sigma, s), "gs_blur_views")
    gs.check(gs.blur_views(src.data_ptr(), out.data_ptr(), _cams(w), 1, k, sigma, s), "gs_blur_views")
    torch.cuda.synchronize()
    assert torch.equal(out[:, :5], ref[:, :5])
    assert torch.allclose(out[:, -5:], ref[:, :5].flip(1), rtol=2 * k * 2.0 ** -24, atol=0)
    for c in range(3):
        lo, hi = out[c, 8 + r:-8 - r].min(), out[c, 8 + r:-8 - r].max()
        assert float(lo) == 0.0 and float(hi) == 0.0
