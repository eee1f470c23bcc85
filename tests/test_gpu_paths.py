"""Edges of the kernels' work splits, on the GPU, against the FP64 oracle or plain references."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2603_09277_amd import gsr, scenes

from gpu_helpers import DEV, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = gsr.Rasterizer(max_views=8)
    yield r
    r.close()


def _cam(w, h):
    return scenes.Camera(w, h, float(w), float(w), w / 2, h / 2, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))


# D-SSIM: bands of 64 pixels, segments of 12 to 124 rows, 32 views a launch.  Tolerances as
# for the plain parity test: FP32 window sums against FP64 (loss absolute, gradient relative L2).
@pytest.mark.parametrize("sizes", [[(63, 12)], [(64, 13), (65, 11)], [(128, 125), (129, 44)], [(1, 130), (200, 1)],
                                   [(7, 9)] * 33 + [(66, 29)]])
@pytest.mark.parametrize("with_grad", [True, False])
def test_dssim_bands_and_segments(R, sizes, with_grad):
    rng = np.random.default_rng(len(sizes) * 100 + sizes[0][0])
    xs = [rng.uniform(0, 1, (h, w, 3)).astype(np.float32) for w, h in sizes]
    ys = [np.clip(x + rng.normal(0, 0.1, x.shape), 0, 1).astype(np.float32) for x in xs]
    x = torch.from_numpy(np.concatenate([a.reshape(-1, 3) for a in xs])).to(DEV)
    y = torch.from_numpy(np.concatenate([a.reshape(-1, 3) for a in ys])).to(DEV)
    grad = torch.zeros_like(x) if with_grad else None
    loss = R.dssim([_cam(w, h) for w, h in sizes], x, y, 0.2, grad).cpu().numpy()
    at = 0
    for v, (w, h) in enumerate(sizes):
        s, gs = orc.ssim(xs[v], ys[v])
        assert abs(loss[v] - 0.2 * (1.0 - s)) <= 2e-5, (v, w, h)
        if with_grad:
            g = grad[at:at + w * h].cpu().numpy().reshape(h, w, 3).astype(np.float64)
            assert np.linalg.norm(g + 0.2 * gs) <= 1e-4 * np.linalg.norm(0.2 * gs), (v, w, h)
        at += w * h


ATTRS = ("means", "scales", "quats", "opacities", "sh")


def _small_scene(n, deg, seed=5):
    scene = scenes.gmm_scene(seed, n, sh_degree=deg, n_clusters=4, box=3.0)
    return scene, {k: v for k, v in to_dev(scene).items()}


# Projection backward: 256 Gaussians a workgroup, 8 views a round, 256 live pairs a pass, the SH
# gradients stored as 16-byte words where they are aligned.  A launch of all views against the sum
# of one-view launches: the same FP32 terms in another order (relative L2 1e-5; SH in BF16: one
# rounding of the sum against a sum of rounded terms, 2^-8 a term).
@pytest.mark.parametrize("n,deg,bf16", [(255, 0, False), (257, 1, False), (300, 1, True), (256, 2, False), (700, 3, False),
                                        (515, 3, True)])
@pytest.mark.parametrize("views,shift", [(2, 0), (9, 0), (17, 1)])
def test_projection_backward_rounds(n, deg, bf16, views, shift):
    scene, t = _small_scene(n, deg)
    if bf16:
        t["sh"] = t["sh"].to(torch.bfloat16)
    opts = gsr.RasterOptions(sh_degree=deg, sh_bf16=bf16)
    cams = scenes.orbit_cameras(np.random.default_rng(views), [(61 + v, 43) for v in range(views)])
    p = [t[k] for k in ATTRS]
    r = gsr.Rasterizer(max_views=views)
    npix = [c.width * c.height for c in cams]
    g_rgb = torch.randn(sum(npix), 3, device=DEV, generator=torch.Generator(DEV).manual_seed(1))
    g_em = torch.full((views,), 0.3, device=DEV)
    grads = {k: torch.full_like(v, 7.0) for k, v in zip(ATTRS, p)}
    # (shift: SH gradients 4 bytes off a 16-byte boundary)
    pad = 4 // t["sh"].element_size() * shift
    grads["sh"] = torch.full((t["sh"].numel() + pad,), 7.0, device=DEV, dtype=t["sh"].dtype)[pad:].view_as(t["sh"])
    out = r.forward(*p, cams, opts)
    got = r.backward(*p, cams, opts, out, g_rgb, None, g_em, grads)
    want = {k: torch.zeros(v.shape, device=DEV, dtype=torch.float64) for k, v in zip(ATTRS, p)}
    at = 0
    for v, cam in enumerate(cams):
        o1 = r.forward(*p, [cam], opts)
        g1 = r.backward(*p, [cam], opts, o1, g_rgb[at:at + npix[v]].contiguous(), None, g_em[v:v + 1])
        at += npix[v]
        for k in ATTRS:
            want[k] += g1[k].double()
    for k in ATTRS:
        d, w = (got[k].double() - want[k]).norm().item(), want[k].norm().item()
        assert w > 0 and d <= (2.0 ** -8 if bf16 and k == "sh" else 1e-5) * w, (k, d / w)
    r.close()


@pytest.mark.parametrize("n", [1, 255, 1025])
def test_pair_counts_of_several_cameras(n):
    scene, t = _small_scene(n, 1)
    opts = gsr.RasterOptions(sh_degree=1)
    cams = scenes.orbit_cameras(np.random.default_rng(3), [(200, 120), (33, 17), (640, 480)])
    p = [t[k] for k in ATTRS]
    r = gsr.Rasterizer(max_views=3)
    r.forward(*p, cams, opts)
    want, tt = r.stats(3)["pairs_per_view"], r.inspect(gsr.BUF_TILES_TOUCHED)
    assert r.pair_counts(*p, cams, opts) == want
    assert np.array_equal(r.inspect(gsr.BUF_TILES_TOUCHED), tt)      # the records of every view
    # r_max: each factor's mean list length, and the last factor's records
    _, means = r.select_rmax(*p, cams[2], opts, 5, 1e-9)
    last = r.inspect(gsr.BUF_TILES_TOUCHED)
    for k in range(1, 6):
        cam = gsr.scaled_camera(cams[2], k)
        (cnt,) = r.pair_counts(*p, [cam], opts)
        assert means[k - 1] == cnt / (-(-cam.width // 16) * -(-cam.height // 16))
    assert np.array_equal(last, r.inspect(gsr.BUF_TILES_TOUCHED))
    r.close()


def _bits(t):
    return t.contiguous().view(torch.int32)


STATS = ("pairs", "evals_fwd", "evals_bwd", "blended", "tested_fwd", "tested_bwd")


# The blend's slotted form (few 8x8 blocks) against the plain form, which the same view takes
# beside a view of 26,600 blocks: 4x4 blocks, 8x8 blocks and tiles cut by the image, one batch
# (256 entries) and window (64) and several, rays that stop, infinite colours, empty tiles.
# Forward outputs and work counts are equal bit by bit; gradients sum the same FP32 terms in another
# order (relative L2 1e-5).
@pytest.mark.parametrize("tile", [(16, 16), (8, 8), (32, 8)])
@pytest.mark.parametrize("size,n,scale", [((1, 1), 40, 1.0), ((5, 3), 300, 3.0), ((33, 31), 63, 1.0), ((33, 31), 700, 2.0),
                                          ((64, 48), 3000, 4.0), ((203, 117), 500, 0.5)])
def test_slotted_blend_equals_plain(tile, size, n, scale):
    scene, t = _small_scene(n, 1)
    t["scales"] = t["scales"] * scale
    if n == 700:
        t["sh"][::97] = 3e38                  # colours that overflow
    (cam,) = scenes.orbit_cameras(np.random.default_rng(8), [size])
    (big,) = scenes.orbit_cameras(np.random.default_rng(9), [(1600, 1060)])
    opts = gsr.RasterOptions(tile=tile, lds_batch=64, sh_degree=1)
    p = [t[k] for k in ATTRS]
    m, mb = cam.width * cam.height, big.width * big.height
    gen = torch.Generator(DEV).manual_seed(4)
    g_rgb, g_h = torch.randn(m, 3, device=DEV, generator=gen), torch.randn(m, device=DEV, generator=gen)
    g_em = torch.full((1,), 0.3, device=DEV)
    r = gsr.Rasterizer(max_views=2)
    out = r.forward(*p, [cam], opts)
    one = {k: out[k].clone() for k in ("rgb", "entropy", "t_final", "n_contrib", "entropy_mean")}
    got = r.backward(*p, [cam], opts, out, g_rgb, g_h, g_em)
    st = r.stats(1)
    image = r.render_image(*p, [cam], opts)
    # the plain form: both views, and the large one alone for its work counts
    out = r.forward(*p, [cam, big], opts)
    zeros = torch.zeros(mb, 3, device=DEV)
    want = r.backward(*p, [cam, big], opts, out, torch.cat([g_rgb, zeros]), torch.cat([g_h, zeros[:, 0]]),
                      torch.cat([g_em, 0 * g_em]))
    both = r.stats(2)
    ob = r.forward(*p, [big], opts)
    r.backward(*p, [big], opts, ob, zeros, zeros[:, 0].contiguous(), 0 * g_em)
    alone = r.stats(1)
    for k in ("rgb", "entropy", "t_final", "n_contrib"):
        assert torch.equal(_bits(one[k]), _bits(out[k][:m])), k
    assert torch.equal(_bits(image), _bits(one["rgb"]))
    assert torch.equal(_bits(one["entropy_mean"]), _bits(out["entropy_mean"][:1]))
    assert {k: st[k] for k in STATS} == {k: both[k] - alone[k] for k in STATS}
    if n != 700:
        for k in ATTRS:
            d, w = (got[k].double() - want[k].double()).norm().item(), want[k].double().norm().item()
            assert d <= 1e-5 * w, (k, d, w)
    r.close()


# Binning: one workgroup up to 6,144 records (1,024 threads, whole rounds and remainders), the
# radix passes beyond; equal depths, one depth for all.  Every tile's list holds each record
# once per tile it touches, in (depth, index) order.
@pytest.mark.parametrize("n", [1, 63, 65, 1023, 1024, 1025, 4097, 6143, 6144, 6145])
@pytest.mark.parametrize("depths", ["all", "few", "one"])
def test_lists_of_few_records(n, depths):
    scene, t = _small_scene(n, 0)
    if depths != "all":
        t["means"][:] = t["means"][torch.arange(n, device=DEV) % (7 if depths == "few" else 1)].clone()
    cams = scenes.orbit_cameras(np.random.default_rng(8), [(150, 70)])
    r = gsr.Rasterizer(max_views=1)
    r.forward(*[t[k] for k in ATTRS], cams, gsr.RasterOptions(sh_degree=0))
    vals, ranges = r.inspect(gsr.BUF_PAIR_VALUES).astype(np.int64), r.inspect(gsr.BUF_RANGES).reshape(-1, 2).astype(np.int64)
    tt, depth = r.inspect(gsr.BUF_TILES_TOUCHED), r.inspect(gsr.BUF_DEPTH)
    assert len(vals) == tt.sum() == (ranges[:, 1] - ranges[:, 0]).sum()
    assert np.array_equal(np.bincount(vals, minlength=n), tt)
    for a, b in ranges:
        order = np.lexsort((vals[a:b], depth[vals[a:b]]))
        assert np.array_equal(order, np.arange(b - a)) and len(set(vals[a:b])) == b - a
    r.close()


# Tile ids of 8 bits (one pass), 16 bits (two) and more (three); pair counts of small and of
# large passes (2^21 pairs), records past one workgroup.  Every list is in (depth, index)
# order and each view's outputs are those of the view alone, whose ids may be narrower.
@pytest.mark.parametrize("sizes", [[(128, 128)], [(128, 128), (8, 8)], [(2048, 2048)], [(8, 8), (2048, 2048)],
                                   [(2048, 2048), (120, 136), (1024, 8)]])
@pytest.mark.parametrize("n,scale", [(700, 1.0), (9000, 1.0), (9000, 6.0)])
def test_tile_sort_key_widths(sizes, n, scale):
    scene, t = _small_scene(n, 0)
    t["scales"] = t["scales"] * scale
    cams = scenes.orbit_cameras(np.random.default_rng(8), sizes)
    opts = gsr.RasterOptions(tile=(8, 8), sh_degree=0)
    p = [t[k] for k in ATTRS]
    r = gsr.Rasterizer(max_views=len(cams))
    out = {k: v.clone() for k, v in r.forward(*p, cams, opts).items() if k in ("rgb", "t_final", "n_contrib")}
    vals, ranges = r.inspect(gsr.BUF_PAIR_VALUES).astype(np.int64), r.inspect(gsr.BUF_RANGES).reshape(-1, 2).astype(np.int64)
    tt, depth = r.inspect(gsr.BUF_TILES_TOUCHED), r.inspect(gsr.BUF_DEPTH)
    ln = ranges[:, 1] - ranges[:, 0]
    assert len(vals) == tt.sum() == ln.sum()
    assert np.array_equal(np.bincount(vals, minlength=n * len(cams)), tt)
    assert np.array_equal(ranges[ln > 0, 0], np.cumsum(ln)[ln > 0] - ln[ln > 0])
    tile = np.repeat(np.arange(len(ln)), ln)
    same = tile[1:] == tile[:-1]
    d = depth[vals]
    assert np.all(~same | (d[1:] > d[:-1]) | ((d[1:] == d[:-1]) & (vals[1:] > vals[:-1])))
    at = 0
    for cam in cams:
        m = cam.width * cam.height
        one = r.forward(*p, [cam], opts)
        for k, v in out.items():
            assert torch.equal(_bits(v[at:at + m]), _bits(one[k])), (k, cam.width)
        at += m
    r.close()


def _check_lists(r, n, views):
    """Every tile's list in (depth, index) order, each record once per tile it touches."""
    vals, ranges = r.inspect(gsr.BUF_PAIR_VALUES).astype(np.int64), r.inspect(gsr.BUF_RANGES).reshape(-1, 2).astype(np.int64)
    tt, depth = r.inspect(gsr.BUF_TILES_TOUCHED), r.inspect(gsr.BUF_DEPTH)
    ln = ranges[:, 1] - ranges[:, 0]
    assert len(vals) == tt.sum() == ln.sum()
    assert np.array_equal(np.bincount(vals, minlength=n * views), tt)
    tile = np.repeat(np.arange(len(ln)), ln)
    d, same = depth[vals], tile[1:] == tile[:-1]
    assert np.all(~same | (d[1:] > d[:-1]) | ((d[1:] == d[:-1]) & (vals[1:] > vals[:-1])))


# The duplication's workgroups of 256, 1,024 and 2,048 records (from 2^18 and 2^21 records on)
# and the rectangles that travel with the sort (from 2^21 records, up to 256 x 256 tiles a
# view): each view's outputs are those of the view alone.
@pytest.mark.parametrize("n,sizes,tile", [(262_143, [(96, 80)], (16, 16)), (262_144, [(96, 80)], (16, 16)),
                                          (1_048_577, [(640, 360), (320, 200)], (16, 16)),
                                          (1_048_577, [(2048, 64), (64, 2048)], (8, 8)),
                                          (1_048_577, [(2049, 64), (64, 64)], (8, 8)),
                                          (1_048_577, [(64, 64), (64, 2049)], (8, 8))])
def test_duplication_sizes(n, sizes, tile):
    scene, t = _small_scene(n, 0)
    cams = scenes.orbit_cameras(np.random.default_rng(8), sizes)
    opts = gsr.RasterOptions(tile=tile, sh_degree=0)
    p = [t[k] for k in ATTRS]
    r = gsr.Rasterizer(max_views=len(cams))
    out = {k: v.clone() for k, v in r.forward(*p, cams, opts).items() if k in ("rgb", "t_final", "n_contrib")}
    _check_lists(r, n, len(cams))
    at = 0
    for cam in cams if len(cams) > 1 else []:
        m = cam.width * cam.height
        one = r.forward(*p, [cam], opts)
        _check_lists(r, n, 1)
        for k, v in out.items():
            assert torch.equal(_bits(v[at:at + m]), _bits(one[k])), (k, cam.width)
        at += m
    r.close()


# One record over more than 2^20 tiles (the quotient by reciprocal ends there), between small ones.
def test_record_over_a_million_tiles():
    scene, t = _small_scene(130, 0)
    t["scales"][::64] = 40.0
    cams = scenes.orbit_cameras(np.random.default_rng(8), [(8200, 8200)])
    r = gsr.Rasterizer(max_views=1)
    r.forward(*[t[k] for k in ATTRS], cams, gsr.RasterOptions(tile=(8, 8), sh_degree=0))
    tt = r.inspect(gsr.BUF_TILES_TOUCHED)
    assert tt.max() == 1025 * 1025 and len(np.unique(tt)) > 3
    _check_lists(r, 130, 1)
    r.close()


# The forward slotted, the backward plain (from 2^20 records on) against both slotted, the
# same Gaussians with and without others far away.
def test_backward_form_by_records():
    n, extra = 3000, 1 << 20
    scene, t = _small_scene(n, 0)
    far = {k: v[:1].expand(extra, *v.shape[1:]) for k, v in t.items()}
    far["means"] = far["means"] + 1e4
    cams = scenes.orbit_cameras(np.random.default_rng(8), [(70, 50)])
    opts = gsr.RasterOptions(sh_degree=0)
    gen = torch.Generator(DEV).manual_seed(4)
    g_rgb, g_h = torch.randn(3500, 3, device=DEV, generator=gen), torch.randn(3500, device=DEV, generator=gen)
    r = gsr.Rasterizer(max_views=1)
    res = []
    for p in ([t[k] for k in ATTRS], [torch.cat([t[k], far[k]]).contiguous() for k in ATTRS]):
        out = r.forward(*p, cams, opts)
        g = r.backward(*p, cams, opts, out, g_rgb, g_h, torch.full((1,), 0.3, device=DEV))
        res.append(({k: out[k].clone() for k in ("rgb", "entropy", "t_final", "n_contrib")}, {k: v[:n] for k, v in g.items()}))
    for k in res[0][0]:
        assert torch.equal(_bits(res[0][0][k]), _bits(res[1][0][k])), k
    for k in ATTRS:
        a, b = res[0][1][k].double(), res[1][1][k].double()
        assert (a - b).norm() <= 1e-5 * a.norm(), k
    r.close()


# The mixed forward (the 128 longest tiles slotted, the rest plain) against the plain one: the
# same view beside another that makes the launch too large for it.
@pytest.mark.parametrize("tile,size", [((16, 16), (597, 397)), ((8, 8), (367, 361)), ((32, 8), (641, 300))])
@pytest.mark.parametrize("n,scale,lds", [(2500, 1.0, 64), (3000, 4.0, 32), (3000, 2.0, 256), (3000, 3.0, 128)])
def test_mixed_blend_equals_plain(tile, size, n, scale, lds):
    scene, t = _small_scene(n, 1)
    t["scales"] = t["scales"] * scale
    (cam,) = scenes.orbit_cameras(np.random.default_rng(8), [size])
    (big,) = scenes.orbit_cameras(np.random.default_rng(9), [(1600, 1060)])
    opts = gsr.RasterOptions(tile=tile, lds_batch=lds, sh_degree=1)
    p = [t[k] for k in ATTRS]
    m = cam.width * cam.height
    r = gsr.Rasterizer(max_views=2)
    out = r.forward(*p, [cam], opts)
    one = {k: out[k].clone() for k in ("rgb", "entropy", "t_final", "n_contrib", "entropy_mean")}
    st = r.stats(1)
    image = r.render_image(*p, [cam], opts)
    out = r.forward(*p, [cam, big], opts)
    both = r.stats(2)
    r.forward(*p, [big], opts)
    alone = r.stats(1)
    for k in ("rgb", "entropy", "t_final", "n_contrib"):
        assert torch.equal(_bits(one[k]), _bits(out[k][:m])), k
    assert torch.equal(_bits(image), _bits(one["rgb"]))
    assert torch.equal(_bits(one["entropy_mean"]), _bits(out["entropy_mean"][:1]))
    fwd = ("evals_fwd", "blended", "tested_fwd")
    assert {k: st[k] for k in fwd} == {k: both[k] - alone[k] for k in fwd}
    r.close()


# The same beyond 2^20 Gaussians, where several views' live pairs are compacted.
@pytest.mark.parametrize("deg,bf16,views", [(0, False, 2), (1, True, 9), (3, False, 3)])
def test_projection_backward_compacted(deg, bf16, views):
    n = (1 << 20) + 513
    scene, t = _small_scene(n, deg)
    if bf16:
        t["sh"] = t["sh"].to(torch.bfloat16)
    opts = gsr.RasterOptions(sh_degree=deg, sh_bf16=bf16)
    cams = scenes.orbit_cameras(np.random.default_rng(views), [(61 + v, 43) for v in range(views)])
    p = [t[k] for k in ATTRS]
    r = gsr.Rasterizer(max_views=views)
    npix = [c.width * c.height for c in cams]
    g_rgb = torch.randn(sum(npix), 3, device=DEV, generator=torch.Generator(DEV).manual_seed(1))
    g_em = torch.full((views,), 0.3, device=DEV)
    got = r.backward(*p, cams, opts, r.forward(*p, cams, opts), g_rgb, None, g_em)
    want = {k: torch.zeros(v.shape, device=DEV, dtype=torch.float64) for k, v in zip(ATTRS, p)}
    at = 0
    for v, cam in enumerate(cams):
        o1 = r.forward(*p, [cam], opts)
        g1 = r.backward(*p, [cam], opts, o1, g_rgb[at:at + npix[v]].contiguous(), None, g_em[v:v + 1])
        at += npix[v]
        for k in ATTRS:
            want[k] += g1[k].double()
    for k in ATTRS:
        d, w = (got[k].double() - want[k]).norm().item(), want[k].norm().item()
        assert w > 0 and d <= (2.0 ** -8 if bf16 and k == "sh" else 1e-5) * w, (k, d / w)
    r.close()


# A replay after a pair count, whose rectangles are the wider words: the tile counts of the frame.
def test_replay_after_pair_counts():
    n = 1 << 21
    scene, t = _small_scene(n, 0)
    cams = scenes.orbit_cameras(np.random.default_rng(8), [(64, 48)])
    opts = gsr.RasterOptions(sh_degree=0, flags=gsr.GSR_DEFAULT_FLAGS | gsr.GSR_GRAPH)
    p = [t[k] for k in ATTRS]
    r = gsr.Rasterizer(max_views=1)
    out = r.forward(*p, cams, opts)
    want = r.inspect(gsr.BUF_TILES_TOUCHED)
    count = r.pair_counts(*p, cams, opts)
    assert count == [want.sum()] and np.array_equal(r.inspect(gsr.BUF_TILES_TOUCHED), want)
    for _ in range(2):
        out = r.forward(*p, cams, opts, out)
        assert np.array_equal(r.inspect(gsr.BUF_TILES_TOUCHED), want)
        _check_lists(r, n, 1)
    r.close()
