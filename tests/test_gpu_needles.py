"""Position gradients of needles: elongated Gaussians whose conic nearly cancels along their length,
against sums in 64 bits of what the backward walk stages."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2501_14534_amd import scenes

K_Q = np.float32(-0.5) * np.float32(1.44269504088896341)  # exponent of 2 per unit of q
ALPHA_MIN, ALPHA_MAX = 1.0 / 255.0, 0.99


def needles(n: int, length: float, seed: int, px: int = 128):
    """n faint Gaussians at random angles on one view, 0.55 pixels across (the low-pass alone) and
    about `length` along."""
    wl = scenes.tiny(n=n, seed=seed, deg=0, width=px, height=px, opacity=(-3.5, 0.3), spread=0.6, depth=(3.0, 4.0))
    sc = wl.scene.copy()
    sc.log_scales[:] = -9.0
    sc.log_scales[0] = np.log(length * 3.5 / px)
    sc.sh_dc[:] = np.abs(sc.sh_dc) + 0.2
    return dataclasses.replace(wl, scene=sc)


def fma32(x, y, z):
    """x y + z rounded once to float (the product of two floats is exact in 64 bits)."""
    return (x.astype(np.float64) * y + z).astype(np.float32)


def rows64(rec, ids, ranges, tw, th, tiles_x, W, H, dL, sum_rows):
    """Per list entry of each tile: sum_rows(m, a dx, b/2 dy, b/2 dx, c dy) over the tile's pixels, for
    the staged conic (a, b, c) and m = alpha dL/dalpha in 64 bits, from the offsets and the exponent as the
    walk rounds them (an exponent's error moves m by as much as any order of the sum).  No pixel stops
    (faint records)."""
    out = []
    for t, (s, e) in enumerate(ranges):
        ty, tx = divmod(t, tiles_x)
        y, x = np.meshgrid(np.arange(th) + ty * th, np.arange(tw) + tx * tw, indexing="ij")
        keep = (x < W) & (y < H)
        x, y = x[keep].astype(np.int64), y[keep].astype(np.int64)
        g = dL[:, y, x].astype(np.float64)
        r = rec[ids[s:e]]
        dx = (x[None] + 0.5).astype(np.float32) - r[:, 0:1]
        dy = (y[None] + 0.5).astype(np.float32) - r[:, 1:2]
        a, b, c = K_Q * r[:, 2:3], (np.float32(2) * K_Q) * r[:, 3:4], K_Q * r[:, 4:5]
        ex = fma32(dx, fma32(b, dy, a * dx), (c * dy) * dy)
        alpha = r[:, 5:6] * np.exp2(ex.astype(np.float64))
        dx, dy, a, hb, c = (v.astype(np.float64) for v in (dx, dy, a, np.float32(0.5) * b, c))
        use = (np.abs(dx) <= r[:, 6:7]) & (np.abs(dy) <= r[:, 6:7]) & (alpha >= ALPHA_MIN)
        alpha = np.where(use, alpha, 0.0)
        assert alpha.size == 0 or alpha.max() < ALPHA_MAX
        T = np.cumprod(1.0 - alpha, 0) / (1.0 - alpha)  # in front of each entry
        cd = r[:, 8:11].astype(np.float64) @ g
        w = alpha * T * cd
        behind = w.sum(0)[None] - np.cumsum(w, 0)  # background 0
        m = np.where(use, alpha * (T * cd - behind / (1.0 - alpha)), 0.0)
        for i in range(e - s):
            out.append(sum_rows(m[i], a[i] * dx[i], hb[i] * dy[i], hb[i] * dx[i], c[i] * dy[i]))
    return np.array(out)


def sums(m, adx, hbdy, hbdx, cdy):
    """The row's (u, v) in units of 1 / kQ, and the root of the summed squares of the pixels' products:
    u, v, |.|_u, |.|_v, pixels."""
    return ((m * (adx + hbdy)).sum(), (m * (hbdx + cdy)).sum(), np.sqrt((m * m * (adx * adx + hbdy * hbdy)).sum()),
            np.sqrt((m * m * (hbdx * hbdx + cdy * cdy)).sum()), (m != 0).sum())


def errors(uv, ref):
    """Error of each row's (u, v) over 2^-24 times the root of its summed squared products, for rows of
    at least 24 pixels."""
    k = ref[:, 4] >= 24
    assert k.sum() >= 100
    return np.abs(uv[k].astype(np.float64) * float(K_Q) - ref[k, 0:2]) / (2.0 ** -24 * ref[k, 2:4])


@pytest.mark.gpu
@pytest.mark.parametrize("length", [10.0, 30.0])
@pytest.mark.parametrize("tw,th,ppt", [(16, 16, 1), (32, 16, 2), (32, 32, 4)])
def test_needle_rows_are_as_accurate_as_their_products(length, tw, th, ppt):
    """Each pixel's m (a dx + b/2 dy) rounds one product before the terms cancel: independent errors of
    at most 2^-24 of it, whose sum has a deviation of at most 1 / sqrt(3) (uniform roundings) of 2^-24 times
    the root of the summed squares: half of the rows within 0.39 of that.  Alpha, the transmittance, the
    colour behind and the sums round terms that have cancelled; with as much again for them 0.55, and
    twice that is allowed.  Sums of m dx and m dy rounded before the conic is applied err by a part of
    the sum itself, not of its root: a median of 1.9 to 3.1."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import parity as P
    wl = needles(int(2000 / length), length, seed=3)
    opts = dataclasses.replace(wl.opts, tile_w=tw, tile_h=th, pixels_per_thread=ppt)
    W, H = wl.cams[0].width, wl.cams[0].height
    dL = np.ones((3, H, W), np.float32)
    print(f"[needles] length {length} tile {tw}x{th} ppt {ppt}", flush=True)
    r, _ = P.gpu_forward(wl, opts)
    assert float(r.T_final.min()) > 1e-3
    rows = r.grad_pairs(torch.from_numpy(dL).cuda().reshape(-1)).cpu().numpy()
    L = P.gpu_lists(r)
    pair = r.pair_index[: L["K"]].cpu().numpy().view(np.uint32)
    ref = rows64(r.splat_records().cpu().numpy(), L["ids"], L["ranges"], tw, th, -(-W // tw), W, H, dL, sums)
    order = np.concatenate([np.arange(s, e) for s, e in L["ranges"]])
    med = np.median(errors(rows[pair[order]][:, 0:2], ref))
    print(f"[needles] median error {med:.3f}", flush=True)
    assert med <= 1.1
