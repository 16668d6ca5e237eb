"""The volume quantile of the significance score (GPU only): counts around a workgroup and around four
rounds of the whole grid, equal keys, keys that differ in one digit alone."""
import numpy as np
import pytest
import torch

from paper_2501_14534_amd import raster

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2501_14534_amd import gs
    gs.load()


@pytest.mark.parametrize("n", [1, 2, 255, 1023, 1024, 1025, 262144, 262145, 1048577])
@pytest.mark.parametrize("kind", ["random", "equal", "low digit"])
def test_score_uses_the_exact_quantile(n, kind):
    """With one hit and opacity 1/2 each, the score is exp(min(lv - lv_q, 0)) / 2: 1/2 exactly for the
    Gaussians at and above the quantile, whose number is known from sorting."""
    rng = np.random.default_rng(n)
    ls = np.zeros((3, n), np.float32)
    if kind == "random":
        ls[:] = rng.standard_normal((3, n)).astype(np.float32) * 2.0 - 4.0
    elif kind == "low digit":
        ls[0] = (np.full(n, np.float32(-3.0).view(np.uint32)) + rng.integers(0, 256, n).astype(np.uint32)).view(np.float32)
    print(f"[select] n {n} {kind}", flush=True)
    params = {"log_scales": torch.from_numpy(ls).cuda(), "opacity_logits": torch.zeros(n, device="cuda")}
    hits = torch.ones(n, dtype=torch.int32, device="cuda")
    got = raster.significance(params, hits, 0.9).cpu().numpy()
    lv = (ls[0] + ls[1]) + ls[2]
    q = np.sort(lv)[int(np.ceil(0.9 * n)) - 1]
    assert (got[lv >= q] == np.float32(0.5)).all()
    ref = 0.5 * np.exp(np.minimum(lv.astype(np.float64) - q, 0.0))
    assert (np.abs(got - ref) <= 4e-6 * ref).all()  # one exponential of |x| < 40: 40 x 2^-24, and its own error
