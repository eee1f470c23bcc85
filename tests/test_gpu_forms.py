"""Kernel forms, and the state of a context across modes, on the GPU, against plain mode, another form or the FP64 oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2603_09277_amd import gsr, scenes

from gpu_helpers import DEV, KEYS, check_grad2d, gpu_records, oracle_stagewise, to_dev

pytestmark = pytest.mark.gpu

IMAGES = ("rgb", "entropy", "t_final", "n_contrib")


def _scene(n, deg=0, scale=1.0, seed=5):
    t = to_dev(scenes.gmm_scene(seed, n, sh_degree=deg, n_clusters=4, box=3.0))
    t["scales"] *= scale
    return t, [t[k] for k in KEYS]


def _cams(*sizes):
    return scenes.orbit_cameras(np.random.default_rng(8), list(sizes))


def _upstream(cams, seed=4):
    m = sum(c.width * c.height for c in cams)
    gen = torch.Generator(DEV).manual_seed(seed)
    return (torch.randn(m, 3, device=DEV, generator=gen), torch.randn(m, device=DEV, generator=gen),
            torch.full((len(cams),), 0.3, device=DEV))


def _near(got, want, tol=1e-5):
    for k in KEYS:
        d, w = (got[k].double() - want[k].double()).norm().item(), want[k].double().norm().item()
        assert w > 0 and d <= tol * w, (k, d, w)


# --------------------------------------------------------------------------- #
# graph replays between eager frames
# --------------------------------------------------------------------------- #

GRAPH = gsr.GSR_DEFAULT_FLAGS | gsr.GSR_GRAPH


def _plain_grads(p, cams, up):
    r = gsr.Rasterizer(max_views=1)
    opts = gsr.RasterOptions(sh_degree=0)
    g = r.backward(*p, cams, opts, r.forward(*p, cams, opts), *up)
    torch.cuda.synchronize()
    r.close()
    return g


# A replayed frame's backward works on that frame's pairs, whatever an eager render on the
# same context held in between: with fewer pairs (the backward must not refuse the frame),
# and with the backward's graph captured at the smaller frame (it must not keep its size).
# Gradients as in plain mode (the same FP32 terms, at most in another order: relative L2 1e-5).
def test_replay_after_renders_of_other_sizes():
    t, p = _scene(8000, scale=2.0)
    cams, small = _cams((300, 200)), _cams((160, 112))      # (too many tiles for a bounded frame)
    up = _upstream(cams)
    gopts, opts = gsr.RasterOptions(sh_degree=0, flags=GRAPH), gsr.RasterOptions(sh_degree=0)
    want = _plain_grads(p, cams, up)
    r = gsr.Rasterizer(max_views=1)
    out = r.forward(*p, cams, gopts)
    grads = {k: torch.empty_like(v) for k, v in t.items()}
    for view in (small, cams, small):
        r.render_image(*p, view, opts)
        out = r.forward(*p, cams, gopts, out)
        _near(r.backward(*p, cams, gopts, out, *up, grads), want)
    r.close()


def test_backward_graph_captured_at_a_smaller_frame():
    t, p = _scene(8000, scale=2.0)
    cams = _cams((300, 200))
    up = _upstream(cams)
    gopts, opts = gsr.RasterOptions(sh_degree=0, flags=GRAPH), gsr.RasterOptions(sh_degree=0)
    full = t["scales"].clone()
    r = gsr.Rasterizer(max_views=1)
    out = r.forward(*p, cams, gopts)                       # the capacity of the larger frame
    grads = {k: torch.empty_like(v) for k, v in t.items()}
    pairs = []
    for scales in (0.3 * full, full, 0.3 * full):
        t["scales"].copy_(scales)
        r.render_image(*p, cams, opts)                     # an eager frame of as many pairs
        out = r.forward(*p, cams, gopts, out)
        got = r.backward(*p, cams, gopts, out, *up, grads)
        _near(got, _plain_grads(p, cams, up))
        pairs.append(r.stats(1)["pairs"])
    assert pairs[0] == pairs[2] < 0.7 * pairs[1]
    r.close()


# --------------------------------------------------------------------------- #
# colours that overflow
# --------------------------------------------------------------------------- #

# An entry with an infinite colour that no pixel blends (opacity 0.006 between the pixel
# centres: it passes the cull, whose rectangle it is over, and reaches 1/255 at none of them)
# has no part in the gradients of the entries around it; the slotted backward takes it in the
# same step as them.  Every gradient is finite and as the plain form's (which the view takes
# beside a large one).
@pytest.mark.parametrize("tile", [(16, 16), (8, 8), (32, 8)])
@pytest.mark.parametrize("place", [0, 1, 3, 6])
def test_infinite_colour_that_no_pixel_blends(tile, place):
    n = 8
    cam = scenes.Camera(16, 16, 16.0, 16.0, 8.0, 8.0, np.eye(3, dtype=np.float32), np.zeros(3, np.float32))
    big = scenes.Camera(1600, 1060, 16.0, 16.0, 8.0, 8.0, cam.R, np.array([0, 0, -100], np.float32))     # sees nothing
    z = 1.0 + torch.arange(n, device=DEV)
    xy = torch.tensor([[0.5 if i % 2 else -2.5, -1.5 + 0.5 * i] for i in range(n)], device=DEV)     # pixels from the centre
    xy[place] = -2.0                                       # inside a 4x4 block
    sh = torch.zeros(n, 9, 3, device=DEV)
    sh[:, 0] = torch.linspace(0.1, 0.8, n, device=DEV)[:, None]
    sh[place, 0::2] = 3.3e38                               # (Y_0, Y_2 and Y_6 are positive along z)
    sh[place, 4] = sh[place, 8] = 0.0
    scale = (3.0 * z / 16.0)[:, None].repeat(1, 3)
    scale[:, 1] *= 0.5
    scale[place] = 1e-4
    p = [torch.cat([xy * z[:, None] / 16.0, z[:, None]], 1).contiguous(), scale,
         torch.tensor([[0.9, 0.1, 0.2, 0.3]], device=DEV).repeat(n, 1),
         torch.full((n,), 0.3, device=DEV), sh]
    p[3][place] = 0.006
    opts = gsr.RasterOptions(tile=tile, sh_degree=2)
    up = _upstream([cam])
    r = gsr.Rasterizer(max_views=2)
    out = r.forward(*p, [cam], opts)
    assert np.isinf(r.inspect(gsr.BUF_RECORDS).reshape(n, 12)[place, 6:9]).all()
    assert torch.isfinite(out["rgb"]).all() and r.stats(1)["tested_fwd"] > 0
    got = r.backward(*p, [cam], opts, out, *up)
    m = big.width * big.height
    zeros = [torch.zeros(m, 3, device=DEV), torch.zeros(m, device=DEV), torch.zeros(1, device=DEV)]
    want = r.backward(*p, [cam, big], opts, r.forward(*p, [cam, big], opts), *(torch.cat(x) for x in zip(up, zeros)))
    for k in KEYS:
        assert torch.isfinite(want[k]).all(), k
        assert torch.isfinite(got[k]).all(), k
    _near(got, want)
    r.close()


# --------------------------------------------------------------------------- #
# frames without host synchronisation
# --------------------------------------------------------------------------- #

# GSR_NO_SYNC frames return while the stream is still busy with earlier work, however many
# views they have (cameras that fit the first kernel's arguments, and more).
@pytest.mark.parametrize("views", [1, 16, 17, 40, 64])
def test_no_sync_returns_before_the_stream(views):
    t, p = _scene(3000)
    cams = _cams(*[(64 + v, 48) for v in range(views)])
    opts = gsr.RasterOptions(sh_degree=0, flags=gsr.GSR_DEFAULT_FLAGS | gsr.GSR_NO_SYNC)
    r = gsr.Rasterizer(max_views=views)
    other = cams[1:] + cams[:1]
    want, want2 = ({k: v.clone() for k, v in r.forward(*p, c, gsr.RasterOptions(sh_degree=0)).items() if k in IMAGES}
                   for c in (cams, other))
    out = r.forward(*p, cams, opts)                        # the mode's first frame sizes the buffers
    a = torch.randn(8192, 8192, device=DEV)
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    for k in IMAGES:
        out[k].zero_()
    out2 = r.forward(*p, other, opts)
    torch.cuda.synchronize()
    end = torch.cuda.Event()
    for _ in range(20):                                    # some 10 ms each
        torch.mm(a, a, out=b)
    end.record()
    out = r.forward(*p, cams, opts, out)
    busy = not end.query()
    out2 = r.forward(*p, other, opts, out2)                # (waits for the frame before: its pair count)
    torch.cuda.synchronize()
    for k in IMAGES:
        assert torch.equal(out[k], want[k]) and torch.equal(out2[k], want2[k]), k
    assert busy
    r.close()


# --------------------------------------------------------------------------- #
# options that a form does not look at
# --------------------------------------------------------------------------- #

# Few blocks, more than 2^20 records: the forward is slotted, the backward is not and takes
# persistent scheduling and lds_batch from the options.
def test_persistent_backward_after_slotted_forward():
    n, extra = 3000, 1 << 20
    t, _ = _scene(n)
    far = {k: v[:1].expand(extra, *v.shape[1:]) for k, v in t.items()}
    far["means"] = far["means"] + 1e4
    p = [torch.cat([t[k], far[k]]).contiguous() for k in KEYS]
    cams = _cams((70, 50))
    up = _upstream(cams)
    r = gsr.Rasterizer(max_views=1)
    res = []
    for flags in (0, gsr.GSR_PERSISTENT, gsr.GSR_PERSISTENT | gsr.GSR_GRAPH):
        opts = gsr.RasterOptions(sh_degree=0, flags=gsr.GSR_DEFAULT_FLAGS | flags)
        out = r.forward(*p, cams, opts)
        g = r.backward(*p, cams, opts, out, *up)
        for _ in range(2):                                 # (queues start afresh for every backward)
            g = r.backward(*p, cams, opts, out, *up, g)
        torch.cuda.synchronize()
        res.append(({k: out[k].clone() for k in IMAGES}, {k: v.clone() for k, v in g.items()}))
    for img, g in res[1:]:
        for k in IMAGES:
            assert torch.equal(img[k], res[0][0][k]), k
        for k in KEYS:
            assert torch.equal(g[k], res[0][1][k]), k
    r.close()


# Where both passes are slotted, lds_batch and GSR_PERSISTENT change nothing: the autotuner
# leaves them as given.
@pytest.mark.parametrize("lds,flags", [(32, 0), (256, gsr.GSR_PERSISTENT), (128, gsr.GSR_GRAPH)])
def test_autotune_leaves_what_changes_nothing(lds, flags, tmp_path):
    t, p = _scene(2000)
    cams = _cams((96, 64))
    opts = gsr.RasterOptions(lds_batch=lds, sh_degree=0, flags=gsr.GSR_DEFAULT_FLAGS | flags)
    r = gsr.Rasterizer(max_views=1)
    best = r.autotune(*p, cams, opts, str(tmp_path / "tune.txt"))
    assert best.tile in ((8, 8), (16, 16), (32, 8)) and best.lds_batch == lds and best.flags == opts.flags
    assert r.autotune(*p, cams, opts, str(tmp_path / "tune.txt")) == best
    r.close()


# --------------------------------------------------------------------------- #
# the forms of frames past the slotted and mixed forms' limits
# --------------------------------------------------------------------------- #

def _form_scene(long):
    scene, cams = scenes.tiny_scene(41, 8000)
    scene.scales = (scene.scales * np.float32(2.0 if long else 0.5)).astype(np.float32)
    c = cams[0]
    f = 1600.0 / c.width
    big = scenes.Camera(1600, 1060, c.fx * f, c.fy * f, 800.0, 530.0, c.R, c.t)     # 26,600 8x8 blocks
    return scene, [c, big]


# The per-block and the shared form of the blends at every batch, in hardware dispatch and
# persistent, on a small view beside a large one: images and 2D gradients of the small view
# against the oracle on the GPU's own records; the two schedulings bit by bit.
@pytest.mark.parametrize("tile,lds", [((16, 16), 32), ((16, 16), 64), ((16, 16), 128), ((16, 16), 256), ((32, 8), 32),
                                      ((32, 8), 64), ((32, 8), 256), ((8, 8), 32), ((8, 8), 128)])
@pytest.mark.parametrize("long", [False, True])
def test_plain_shared_and_persistent_forms_vs_oracle(tile, lds, long):
    from test_gpu_parity import _cmp_image
    scene, cams = _form_scene(long)
    cam, t = cams[0], to_dev(scene)
    p = [t[k] for k in KEYS]
    m, M = cam.width * cam.height, sum(c.width * c.height for c in cams)
    g_rgb = torch.zeros(M, 3, device=DEV)
    g_rgb[:m] = torch.randn(m, 3, device=DEV, generator=torch.Generator(DEV).manual_seed(1)) / m
    g_em = torch.tensor([0.3, 0.0], device=DEV)
    r = gsr.Rasterizer(max_views=2)
    res = []
    for flags in (0, gsr.GSR_PERSISTENT):
        opts = gsr.RasterOptions(tile=tile, lds_batch=lds, sh_degree=0, flags=gsr.GSR_DEFAULT_FLAGS | flags)
        out = r.forward(*p, cams, opts)
        grads = r.backward(*p, cams, opts, out, g_rgb, None, g_em)
        st = r.stats(2)
        assert (st["mean_len"] >= 256) == long, st["mean_len"]
        res.append(({k: out[k].clone() for k in IMAGES + ("entropy_mean",)}, {k: v.clone() for k, v in grads.items()},
                    r.inspect(gsr.BUF_GRAD2D), st, r.render_image(*p, cams, opts)))
    out, grads, g2, st, image = res[0]
    assert torch.equal(image, out["rgb"]) and torch.equal(res[1][4], out["rgb"])
    for k in out:
        assert torch.equal(res[1][0][k], out[k]), k
    for k in KEYS:
        assert torch.equal(res[1][1][k], grads[k]), k
    assert np.array_equal(res[1][2], g2)
    assert res[1][3] == st
    r.forward(*p, cams, opts)
    pg = gpu_records(r, scene.n, 2)[0]
    img_o = oracle_stagewise(pg, cam, tile)
    _cmp_image(out, img_o, cam, 0, cams)
    g2o = orc.backward_render(cam.width, cam.height, tile[0], tile[1], pg["mean2d"], pg["conic"], pg["opacity"], pg["rgb"],
                              img_o["ranges"], img_o["values"],
                              g_rgb[:m].cpu().numpy().reshape(cam.height, cam.width, 3).astype(np.float64),
                              np.full((cam.height, cam.width), np.float64(np.float32(0.3)) / m))
    check_grad2d(g2.reshape(2, scene.n, 9)[0].astype(np.float64), g2o)
    r.close()


# The dense slotted backward (16x16 and 32x8 tiles, 6,145 to 10,240 blocks, two records a
# block or more): images and work counts equal the plain form's, which the view takes beside a
# large one, bit by bit; the 2D gradients of both are within the oracle's tolerance on the
# GPU's own records (their sums over pixels are in another order).
@pytest.mark.parametrize("tile,size", [((16, 16), (800, 513)), ((16, 16), (1011, 631)), ((32, 8), (803, 509))])
@pytest.mark.parametrize("scale", [1.0, 4.0])
def test_dense_slotted_backward(tile, size, scale):
    n = 21_000
    t, p = _scene(n, 1, scale)
    (cam,), (big,) = _cams(size), scenes.orbit_cameras(np.random.default_rng(9), [(1600, 1060)])
    blocks = -(-size[0] // tile[0]) * -(-size[1] // tile[1]) * 4
    assert 6144 < blocks <= 10240 and n >= 2 * blocks
    opts = gsr.RasterOptions(tile=tile, sh_degree=1)
    up = _upstream([cam])
    m, mb = cam.width * cam.height, big.width * big.height
    zeros = [torch.zeros(mb, 3, device=DEV), torch.zeros(mb, device=DEV), torch.zeros(1, device=DEV)]
    r = gsr.Rasterizer(max_views=2)
    out = r.forward(*p, [cam], opts)
    one = {k: out[k].clone() for k in IMAGES}
    r.backward(*p, [cam], opts, out, *up)
    st, g2 = r.stats(1), r.inspect(gsr.BUF_GRAD2D).reshape(n, 9)
    out = r.forward(*p, [cam, big], opts)
    r.backward(*p, [cam, big], opts, out, *(torch.cat(x) for x in zip(up, zeros)))
    both, g2p = r.stats(2), r.inspect(gsr.BUF_GRAD2D).reshape(2, n, 9)[0]
    pg = gpu_records(r, n, 2)[0]
    r.backward(*p, [big], opts, r.forward(*p, [big], opts), *zeros)
    alone = r.stats(1)
    for k in IMAGES:
        assert torch.equal(one[k], out[k][:m]), k
    for k in ("pairs", "evals_fwd", "evals_bwd", "blended", "tested_fwd", "tested_bwd"):
        assert st[k] == both[k] - alone[k], k
    vals, ranges = orc.bin_lists(pg["mean2d"], pg["radius"], pg["depth32"], cam.width, cam.height, tile[0], tile[1])
    shape = (cam.height, cam.width)
    g2o = orc.backward_render(cam.width, cam.height, tile[0], tile[1], pg["mean2d"], pg["conic"], pg["opacity"], pg["rgb"],
                              ranges, vals, up[0].cpu().numpy().reshape(*shape, 3).astype(np.float64),
                              up[1].cpu().numpy().reshape(shape).astype(np.float64) + np.float64(np.float32(0.3)) / m)
    for g in (g2p, g2):
        check_grad2d(g.astype(np.float64), g2o)
    r.close()


# Tile order and mean entropy in one kernel or in two (from 5,121 tiles and from a view of 20,481 8x8
# blocks on): every tile is served, as without an order (persistent scheduling, bit by bit),
# and L_E is the FP64 mean of the entropy map to FP32 rounding.
@pytest.mark.parametrize("tile,sizes", [((16, 16), [(1280, 1024)]), ((16, 16), [(1296, 1024)]), ((16, 16), [(1920, 1080)]),
                                        ((8, 8), [(1280, 1024)]), ((8, 8), [(1281, 1024)]), ((32, 8), [(1280, 1024), (1281, 1025)])])
def test_one_and_two_kernel_forms(tile, sizes):
    t, p = _scene(7000, scale=2.0)
    cams = _cams(*sizes)
    r = gsr.Rasterizer(max_views=2)
    res = []
    for flags in (0, gsr.GSR_PERSISTENT):
        out = r.forward(*p, cams, gsr.RasterOptions(tile=tile, sh_degree=0, flags=gsr.GSR_DEFAULT_FLAGS | flags), None)
        res.append({k: out[k].clone() for k in IMAGES + ("entropy_mean",)})
    for k in res[0]:
        assert torch.equal(res[0][k], res[1][k]), k
    at = 0
    for v, c in enumerate(cams):
        h = res[0]["entropy"][at:at + c.width * c.height].double().mean().item()
        assert h > 0 and abs(res[0]["entropy_mean"][v].item() - h) <= 2e-6 * h
        at += c.width * c.height
    r.close()


# D-SSIM at sizes between those of one round of short segments and several rounds of long ones;
# tolerances as for the parity test of its bands (FP32 window sums against FP64).
@pytest.mark.parametrize("sizes", [[(320, 480)], [(65, 700)], [(486, 324), (97, 65)], [(20, 2000)]])
def test_dssim_segments_of_mid_sized_images(sizes):
    rng = np.random.default_rng(sizes[0][1])
    xs = [rng.uniform(0, 1, (h, w, 3)).astype(np.float32) for w, h in sizes]
    ys = [np.clip(x + rng.normal(0, 0.1, x.shape), 0, 1).astype(np.float32) for x in xs]
    x, y = (torch.from_numpy(np.concatenate([a.reshape(-1, 3) for a in s])).to(DEV) for s in (xs, ys))
    cams = _cams(*sizes)
    grad = torch.zeros_like(x)
    r = gsr.Rasterizer(max_views=2)
    loss = r.dssim(cams, x, y, 0.2, grad).cpu().numpy()
    at = 0
    for v, (w, h) in enumerate(sizes):
        s, gs = orc.ssim(xs[v], ys[v])
        g = grad[at:at + w * h].cpu().numpy().reshape(h, w, 3).astype(np.float64)
        assert abs(loss[v] - 0.2 * (1.0 - s)) <= 2e-5, (v, w, h)
        assert np.linalg.norm(g + 0.2 * gs) <= 1e-4 * np.linalg.norm(0.2 * gs), (v, w, h)
        at += w * h
    r.close()
