"""Every tile shape that the FP32 launches choose, on images with tiles inside
the image as well as ragged ones at its edges.

The sizes select the shapes on 256 CUs: W is 6 tiles of 256 columns and a
remainder, the heights give more or fewer tiles than the launch rules ask."""
import numpy as np
import pytest

import oracle
import paper_1302_5586_amd as pf
import synth
from gpu_util import U, device, gamma

pytestmark = pytest.mark.gpu

W = 1573


def _t(a, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


# 1317 rows: 2075 tiles of 64 x 16, 581 of 256 x 16, 1050 of 64 x 32. Above 1765
# rows 777 tiles of 256 x 16; above 3941 rows 3100 tiles of 64 x 32.
@pytest.mark.parametrize("h", [1317, 1765, 3941])
@pytest.mark.parametrize("r", range(0, pf.PF_R_MAX + 1))
def test_large_tiles(r, h):
    """2D: 128 x 32 and 256 x 16 (r <= 2), 128 x 16 (r = 3), 64 x 32 above;
    separable: 128 x 32 and 256 x 16 (r <= 3), 128 x 32 above, in exact mode
    from r = 5 on 64 x 32 and 64 x 64. Exact mode bit for bit the oracle, both
    modes bit for bit the strip kernel."""
    dev = device()
    rng = np.random.default_rng(7000 + 10 * r + h)
    img = rng.standard_normal((h, W)).astype(np.float32)
    img.flat[rng.integers(0, img.size)] = np.inf
    x = _t(img, dev)
    with np.errstate(invalid="ignore"):
        if h < 3941:  # 2D shapes change with the first two heights only
            f = rng.standard_normal((2 * r + 1, 2 * r + 1)).astype(np.float32)
            fd = _t(f, dev)
            for exact in (False, True):
                got = pf.filter2d(x, fd, exact=exact).cpu().numpy()
                strip = pf.filter_shaped(x, fd, r, pf.KIND_2D, pf.VAR_DIRECT, 32, 4, exact=exact).cpu().numpy()
                assert np.array_equal(got, strip, equal_nan=True), "2d exact=%d" % exact
            assert np.array_equal(got, oracle.filter2d_f32(img, f), equal_nan=True)
        fx, fy = rng.standard_normal((2, 2 * r + 1)).astype(np.float32)
        fxd, fyd, f2 = _t(fx, dev), _t(fy, dev), _t(np.concatenate([fx, fy]), dev)
        for exact in (False, True):
            got = pf.filter_sep(x, fxd, fyd, exact=exact).cpu().numpy()
            strip = pf.filter_shaped(x, f2, r, pf.KIND_SEP, pf.VAR_SEPARABLE, 32, 4, exact=exact).cpu().numpy()
            assert np.array_equal(got, strip, equal_nan=True), "sep exact=%d" % exact
        assert np.array_equal(got, oracle.filter_sep_f32(img, fx, fy), equal_nan=True)


@pytest.mark.parametrize("border", [pf.BORDER_ZERO, pf.BORDER_REFLECT, pf.BORDER_MIRROR])
@pytest.mark.parametrize("r,h", [(1, 1317), (2, 1765), (3, 1317), (8, 1317)])
def test_large_tiles_under_border_rules(r, h, border):
    dev = device()
    rng = np.random.default_rng(7500 + r + border)
    img = rng.standard_normal((h, W)).astype(np.float32)
    f = rng.standard_normal((2 * r + 1, 2 * r + 1)).astype(np.float32)
    got = pf.filter2d_border(_t(img, dev), _t(f, dev), border, exact=True).cpu().numpy()
    assert np.array_equal(got, oracle.filter2d_f32_border(img, f, border))


# 533 columns: 245 rows are 272 tiles of 32 x 16 and 144 of 64 x 16, 899 rows
# 513 of 64 x 16. Neither has rows enough for streams.
@pytest.mark.parametrize("border", [pf.BORDER_CLAMP, pf.BORDER_ZERO, pf.BORDER_REFLECT, pf.BORDER_MIRROR])
@pytest.mark.parametrize("r,passes", [(0, 3), (1, 16), (2, 3), (3, 5), (4, 2), (4, 4), (5, 3), (8, 2)])
def test_chain_tile_forms(r, passes, border):
    """Chains on tiles of 64 x 16 and of 64 x 32: exact mode bit for bit the
    oracle at every pass; the default mode within the relative error that one
    pass may have (gpu_util), once per pass, on non-negative data."""
    dev = device()
    rng = np.random.default_rng(7700 + 100 * r + 10 * passes + border)
    f = synth.gaussian_2d(r, 1.3)
    rel = 1e-5 if r <= 4 else 2 * gamma((2 * r + 1) ** 2) + U
    for h in (245, 899):
        img = rng.random((h, 533), dtype=np.float32)
        x, fd = _t(img, dev), _t(f, dev)
        ref = oracle.filter_chain_f32(img, f, passes, border)
        got = pf.filter_chain(x, fd, passes, border, exact=True).cpu().numpy()
        assert np.array_equal(got, ref), h
        fma = pf.filter_chain(x, fd, passes, border).cpu().numpy().astype(np.float64)
        assert np.all(np.abs(fma - ref) <= passes * rel * (1 + 1e-3) * np.abs(ref) + 1e-30), h


@pytest.mark.parametrize("h,w", [(1, 1), (1, 3), (2, 2), (1, 4099), (5, 3277), (16385, 1), (1027, 1029)])
def test_radius_0(h, w):
    """Radius 0, where a pixel meets one weight per pass: ends of vectors and
    of workgroups, rows off 16-byte alignment, every border rule. The oracle's
    values in both modes: with nothing to add, a fused multiply-add rounds once
    as the multiplication does."""
    dev = device()
    import torch
    rng = np.random.default_rng(7900 + h)
    img = rng.standard_normal((h, w)).astype(np.float32)
    img.flat[0] = np.inf
    f, g = np.array([[-1.7]], np.float32), np.array([[0.3]], np.float32)
    buf = torch.zeros(h * w + 1, device=dev)
    x = buf[1:].view(h, w)
    x.copy_(_t(img, dev))
    fd, gd = _t(f, dev), _t(g, dev)
    for exact in (False, True):
        out = torch.full((h * w + 2,), 7.0, device=dev)
        pf.filter2d(x, fd, exact=exact, out=out[1:-1].view(h, w))
        got = out.cpu().numpy()
        assert np.array_equal(got[1:-1].reshape(h, w), oracle.filter2d_f32(img, f)) and got[0] == got[-1] == 7.0
        assert np.array_equal(pf.filter_sep(x, fd[0], gd[0], exact=exact).cpu().numpy(),
                              oracle.filter_sep_f32(img, f[0], g[0]))
        for border in (pf.BORDER_CLAMP, pf.BORDER_ZERO, pf.BORDER_REFLECT, pf.BORDER_MIRROR):
            for passes in (1, 5, 40):
                assert np.array_equal(pf.filter_chain(x, gd, passes, border, exact=exact).cpu().numpy(),
                                      oracle.filter_chain_f32(img, g, passes, border))


# More than 2048 tiles of 64 x 16 on 256 CUs, thinner than the tile of larger
# images: rows on both sides of the lines to the strip kernel and to 64 x 16
# tiles, columns on 64 x 32 and 128 x 32 tiles.
@pytest.mark.parametrize("h,w", [(3, 131137), (9, 131137), (13, 131137), (16, 131137), (17, 131137), (32785, 5),
                                 (16401, 130), (16401, 100), (7001, 300)])
@pytest.mark.parametrize("r", range(1, pf.PF_R_MAX + 1))
def test_thin_images(r, h, w):
    dev = device()
    rng = np.random.default_rng(8000 + 10 * r + h)
    img = rng.standard_normal((h, w)).astype(np.float32)
    f = rng.standard_normal((2 * r + 1, 2 * r + 1)).astype(np.float32)
    fx, fy = rng.standard_normal((2, 2 * r + 1)).astype(np.float32)
    x, fd, fxd, fyd, f2 = (_t(a, dev) for a in (img, f, fx, fy, np.concatenate([fx, fy])))
    for exact in (False, True):
        got, gots = pf.filter2d(x, fd, exact=exact), pf.filter_sep(x, fxd, fyd, exact=exact)
        assert (got == pf.filter_shaped(x, fd, r, pf.KIND_2D, pf.VAR_DIRECT, 16, 2, exact=exact)).all()
        assert (gots == pf.filter_shaped(x, f2, r, pf.KIND_SEP, pf.VAR_SEPARABLE, 16, 2, exact=exact)).all()
    rows = slice(max(0, h // 2 - 8), h // 2 + 9)  # the oracle on a band and its halo, of the columns at both ends
    for cols in (slice(0, 500), slice(max(0, w - 500), w)):
        band = img[max(0, rows.start - r):rows.stop + r, max(0, cols.start - r):cols.stop + r]
        at = (slice(min(rows.start, r), min(rows.start, r) + min(rows.stop, h) - rows.start),
              slice(min(cols.start, r), min(cols.start, r) + min(cols.stop, w) - cols.start))
        assert np.array_equal(got[rows, cols].cpu().numpy(), oracle.filter2d_f32(band, f)[at])
        assert np.array_equal(gots[rows, cols].cpu().numpy(), oracle.filter_sep_f32(band, fx, fy)[at])


@pytest.mark.parametrize("rows", [159, 4])
@pytest.mark.parametrize("kinds", ["2d", "sep", "both"])
@pytest.mark.parametrize("exact", [False, True])
def test_batches_of_small_images(kinds, exact, rows):
    """More images than the chip takes at once, none of which fills a 256 x 20
    tile: tiles of 64 x 32 for images of few columns, of 256 x 4 for images of
    few rows, every radius, sizes at the tiles' edges and drawn. Every image
    equals its single-image call bit for bit."""
    dev = device()
    import torch
    rng = np.random.default_rng(8300)
    if rows == 4:
        sizes = [(1, 1), (2, 3), (3, 255), (4, 256), (4, 257), (5, 40), (1, 4001)]
        sizes += [(int(h), int(w)) for h, w in zip(rng.integers(1, 6, 43), rng.integers(1, 1300, 43))]
    else:
        sizes = [(1, 1), (2, 3), (31, 63), (32, 64), (33, 65), (64, 64), (65, 128), (97, 130)]
        sizes += [(int(h), int(w)) for h, w in rng.integers(1, rows + 1, (52, 2))]
    imgs, filts, ks = [], [], []
    for i, (h, w) in enumerate(sizes):
        for r in range(pf.PF_BATCH_R_MAX + 1):
            sep = kinds == "sep" or (kinds == "both" and (i + r) % 2)
            imgs.append(rng.standard_normal((h, w)).astype(np.float32))
            filts.append(rng.standard_normal(2 * (2 * r + 1) if sep else (2 * r + 1) ** 2).astype(np.float32))
            ks.append(pf.KIND_SEP if sep else pf.KIND_2D)
    pk = pf.pack_batch(imgs, filts, ks)
    cover = lambda th, tw: int((-(-pk.h // th) * -(-pk.w // tw)).sum())
    tiles = cover(4, 256) if rows == 4 else cover(32, 64)
    assert cover(16, 64) > 2048
    x, fl = _t(pk.pixels, dev), _t(pk.filters, dev)
    out = torch.full_like(x, float("nan"))
    plan = pf.BatchPlan(pk.h, pk.w, pk.r, pk.kind, pk.pix_off, pk.filt_off, x.numel(), fl.numel(), exact=exact)
    assert plan.info()["tasks"] == tiles
    assert pf.batch_plan_check(pk.h, pk.w, pk.r, pk.kind, pk.pix_off, pk.filt_off, x.numel(),
                               fl.numel()) == {"tiles": tiles, "violations": 0}
    plan.run(x, fl, out)
    got = out.cpu().numpy()
    used = np.zeros(x.numel(), bool)
    for i, img in enumerate(imgs):
        h, w, r = int(pk.h[i]), int(pk.w[i]), int(pk.r[i])
        span = slice(pk.pix_off[i], pk.pix_off[i] + h * w)
        used[span] = True
        f, k = _t(filts[i], dev), 2 * r + 1
        ref = (pf.filter2d(_t(img, dev), f.reshape(k, k), exact=exact) if ks[i] == pf.KIND_2D else
               pf.filter_sep(_t(img, dev), f[:k].contiguous(), f[k:].contiguous(), exact=exact))
        assert np.array_equal(got[span].reshape(h, w), ref.cpu().numpy()), (h, w, r, ks[i])
    assert np.isnan(got[~used]).all()
    plan.close()


# Rows per band that give the streams the share of useful work they ask for on
# 256 CUs (two strips of columns, 512 bands, the last one short).
@pytest.mark.parametrize("r,passes,by,border", [
    (1, 9, 24, pf.BORDER_CLAMP), (1, 11, 24, pf.BORDER_ZERO), (1, 14, 30, pf.BORDER_REFLECT), (1, 15, 46, pf.BORDER_MIRROR),
    (1, 16, 46, pf.BORDER_CLAMP), (2, 3, 80, pf.BORDER_MIRROR), (2, 5, 56, pf.BORDER_ZERO), (2, 8, 44, pf.BORDER_REFLECT),
    (3, 2, 44, pf.BORDER_CLAMP), (3, 4, 400, pf.BORDER_REFLECT), (3, 5, 40, pf.BORDER_MIRROR)])
def test_chain_streams_of_many_rows(r, passes, by, border):
    """Bands of rows at the top, inside and at the bottom of a large image: exact
    mode bit for bit the oracle, both modes bit for bit the chain of the band
    alone, which runs on tiles."""
    dev = device()
    import torch
    halo = r * passes
    side = 4 * ((halo + 3) // 4)
    h, w = 32 + 512 * by - 3 + halo, 64 + 2 * (256 - 2 * side) + side
    x = torch.rand((h, w), generator=torch.Generator(device=dev).manual_seed(r * 100 + passes), device=dev)
    f = synth.gaussian_2d(r, 1.1)
    fd = _t(f, dev)
    got = {exact: pf.filter_chain(x, fd, passes, border, exact=exact) for exact in (False, True)}
    n = 130
    for y0 in (0, h // 2 // by * by + 7, h - n):
        lo, hi = y0 + (halo if y0 else 0), y0 + n - (halo if y0 + n < h else 0)  # rows the band alone determines
        band = x[y0:y0 + n].contiguous()
        ref = oracle.filter_chain_f32(band.cpu().numpy(), f, passes, border)
        assert np.array_equal(got[True][lo:hi].cpu().numpy(), ref[lo - y0:hi - y0]), y0
        for exact in (False, True):
            assert torch.equal(got[exact][lo:hi], pf.filter_chain(band, fd, passes, border, exact=exact)[lo - y0:hi - y0]), y0


@pytest.mark.parametrize("h,w", [(40, 60001), (100, 33001), (395, 16129), (64, 40193)])
@pytest.mark.parametrize("r", [1, 3, 4, 6])
def test_wide_images(r, h, w):
    """Images of few rows of tiles and many columns, whose tiles are taken in
    panels, the last one ragged: every pixel equals the strip kernel's."""
    dev = device()
    import torch
    g = torch.Generator(device=dev).manual_seed(8500 + r)
    x = torch.randn((h, w), generator=g, device=dev)
    f, k = torch.randn((2 * r + 1, 2 * r + 1), generator=g, device=dev), 2 * r + 1
    for exact in (False, True):
        assert torch.equal(pf.filter2d(x, f, exact=exact),
                           pf.filter_shaped(x, f.ravel(), r, pf.KIND_2D, pf.VAR_DIRECT, 32, 4, exact=exact))
        assert torch.equal(pf.filter_sep(x, f[0], f[1], exact=exact),
                           pf.filter_shaped(x, f[:2].ravel(), r, pf.KIND_SEP, pf.VAR_SEPARABLE, 32, 4, exact=exact))
