"""Autograd gradients of the SH bands and band masks above the degree in use are zero, whatever the
memory they are written into held before (GPU only)."""
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


@pytest.mark.parametrize("deg", [0, 1, 2, 3])
def test_unused_bands_get_zero_gradients(deg):
    n = 300
    wl = scenes.tiny(n=n, seed=9, deg=3, masks=True, band_masks=True)
    params = {k: v.requires_grad_() for k, v in raster.to_device(wl.scene).items() if v is not None}
    r = raster.Rasterizer(n, deg, wl.cams, wl.opts)
    print(f"[bands] degree {deg}", flush=True)
    img = raster.rasterize(r, params)
    junk = [torch.full_like(v, float("nan")) for _ in range(3) for v in params.values()]
    del junk  # the next allocations of these sizes hold NaN
    img.square().sum().backward()
    r2 = raster.Rasterizer(n, deg, wl.cams, wl.opts)
    plain = {k: v.detach() for k, v in params.items()}
    r2.forward(plain)
    ref = r2.zero_grads(plain)
    r2.backward(plain, 2.0 * r2.image, ref)
    for k, v in params.items():
        assert torch.equal(v.grad, ref[k]), k
    assert int((params["sh_mask_logits"].grad[deg:] != 0).sum()) == 0
